// Expert FFN for two or more tokens (apex_moe_ffn, batch >= 2): a grouped GEMM on the
// matrix cores.
//
// up_gemm and down_gemm take tokens as the M dimension (tiles of 16, padded), weight
// rows as N and the hidden / intermediate dimension as K, with v_mfma_f32_16x16x32_bf16
// (activations rounded to bf16, fp32 accumulation).  A workgroup owns 64 weight rows of
// one expert (blockIdx.y is the expert id; experts without a slot exit at once) and
// finds that expert's (token, position) pairs itself from exec_idx, in pair order, while
// its first weight block loads into LDS (an expert without tokens then exits).  When a projection has too few row tiles to keep the chip's loads in flight
// (plan_for), its K range is split over blockIdx.z and each split writes fp32 partial
// sums:
//   * up_gemm with one split writes h = bf16(silu(W1 x) * (W3 x)) per pair; with several
//     it writes the partial W1 x and W3 x, and swiglu_reduce adds them (in split order)
//     into the same bf16 h, once, before down_gemm reads it from every row tile;
//   * down_gemm writes per-split, per-pair outputs; combine_pairs adds the splits and the
//     gated positions of each token in a fixed order.
// Slots hold bf16 weights (apex_pack_expert), E4M3 codes with fp32 row scales
// (apex_pack_expert_fp8) or MXFP4 codes with a power-of-two scale per block of 32
// (apex_pack_expert_mxfp4).  Weights go from memory to LDS as they are stored; E4M3 and
// MXFP4 codes are widened to bf16 exactly at fragment read (MXFP4 with its block scales
// applied); the E4M3 row scales multiply the outputs.  Every executed expert's weights are read once per call
// whatever the number of tokens routed to it, and no atomics are used, so results are
// deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "ffn_device.h"
#include "ffn_internal.h"

namespace {

using apex::ffn::kWave;
using apex::ffn::silu;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kRows = 64;          // weight rows per workgroup tile
constexpr int kMaxSplit = 4;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint4 pack_bf16(float a0, float a1, float a2, float a3, float a4,
                                           float a5, float a6, float a7) {
    bf16x8 v;
    v[0] = (__bf16)a0; v[1] = (__bf16)a1; v[2] = (__bf16)a2; v[3] = (__bf16)a3;
    v[4] = (__bf16)a4; v[5] = (__bf16)a5; v[6] = (__bf16)a6; v[7] = (__bf16)a7;
    return __builtin_bit_cast(uint4, v);
}

// Component-wise select: a select of the whole vector struct is lowered through
// private memory by the compiler.
__device__ __forceinline__ uint4 keep_if(uint4 v, bool c) {
    return make_uint4(c ? v.x : 0u, c ? v.y : 0u, c ? v.z : 0u, c ? v.w : 0u);
}

// Activation sources: 8 consecutive K values of one row.  load() fetches them as they are
// stored and to_bf16() converts them when the block is staged in LDS, so that no
// arithmetic follows a load directly (which would make the compiler wait for it, and for
// every older load, before the matrix cores work on the previous block).
struct ActF32 {          // fp32 rows (the FFN input x), rounded to bf16 at staging
    static constexpr int kLoads = 2;
    struct Raw {
        float4 a, b;
    };
    static __device__ __forceinline__ Raw load(const void *row, int kc) {
        const float4 *p = reinterpret_cast<const float4 *>(static_cast<const float *>(row) + kc);
        return Raw{p[0], p[1]};
    }
    static __device__ __forceinline__ uint4 to_bf16(const Raw &r) {
        return pack_bf16(r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w);
    }
};
struct ActBf16 {         // bf16 rows (h)
    static constexpr int kLoads = 1;
    using Raw = uint4;
    static __device__ __forceinline__ Raw load(const void *row, int kc) {
        return *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(row) + kc);
    }
    static __device__ __forceinline__ uint4 to_bf16(const Raw &r) { return r; }
};
// h = bf16(silu(u) * v) of 8 consecutive values from SU split partials: u of split s at
// r + 2s*stride, v at r + (2s+1)*stride, the splits added in order.
template <int SU>
__device__ __forceinline__ uint4 swiglu8(const float *r, size_t stride) {
    float u[8], v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) u[c] = v[c] = 0.f;
#pragma unroll
    for (int s = 0; s < SU; ++s) {
        const float4 *pu = reinterpret_cast<const float4 *>(r + 2 * s * stride);
        const float4 *pv = reinterpret_cast<const float4 *>(r + (2 * s + 1) * stride);
        const float4 u0 = pu[0], u1 = pu[1], v0 = pv[0], v1 = pv[1];
        u[0] += u0.x; u[1] += u0.y; u[2] += u0.z; u[3] += u0.w;
        u[4] += u1.x; u[5] += u1.y; u[6] += u1.z; u[7] += u1.w;
        v[0] += v0.x; v[1] += v0.y; v[2] += v0.z; v[3] += v0.w;
        v[4] += v1.x; v[5] += v1.y; v[6] += v1.z; v[7] += v1.w;
    }
    return pack_bf16(silu(u[0]) * v[0], silu(u[1]) * v[1], silu(u[2]) * v[2],
                     silu(u[3]) * v[3], silu(u[4]) * v[4], silu(u[5]) * v[5],
                     silu(u[6]) * v[6], silu(u[7]) * v[7]);
}

// Weight formats of a slot.
// kUpGroups: workgroups the gate/up projection's K splits aim at (see plan_for);
// kKPerElem: K values per element of T; kFp8: fp32 row scales after the codes;
// kBlockScale: one scale byte per 32 K values of a row;
// kChunkK: K values in 16 bytes of a row; plan_kb<MT>(): K values that the split rule
// counts as one block.
struct WBf16 {           // apex_pack_expert slots: bf16 weights
    using T = uint16_t;
    static constexpr bool kFp8 = false, kBlockScale = false;
    template <int MT> static constexpr int plan_kb() { return 128; }
    static constexpr int kUpGroups = 400, kKPerElem = 1, kChunkK = 8;
};
struct WE4M3 {           // apex_pack_expert_fp8 slots: E4M3 codes, fp32 row scales after them
    using T = uint8_t;
    static constexpr bool kFp8 = true, kBlockScale = false;
    template <int MT> static constexpr int plan_kb() { return MT == 1 ? 256 : 128; }
    static constexpr int kUpGroups = 800, kKPerElem = 1, kChunkK = 16;
};
struct WMxfp4 {          // apex_pack_expert_mxfp4 slots: two E2M1 codes per byte, block scales
    using T = uint8_t;
    static constexpr bool kFp8 = false, kBlockScale = true;
    template <int MT> static constexpr int plan_kb() { return MT == 1 ? 512 : 256; }
    static constexpr int kUpGroups = 1400, kKPerElem = 2, kChunkK = 32;
};

constexpr int kPairRounds = APEX_MAX_PAIRS / kThreads;

// This thread's exec_idx entries, pairs r * 256 + t (the index clamped to P - 1; entries
// past P are dropped by expert_pairs).  Issued before a tile's first weight loads, so
// that the pair scan waits only for these, not for the weights.
__device__ __forceinline__ void pair_ids(const int32_t *__restrict__ exec_idx, int P,
                                         int (&ev)[kPairRounds]) {
#pragma unroll
    for (int r = 0; r < kPairRounds; ++r) {
        const int p = r * kThreads + threadIdx.x;
        ev[r] = r == 0 || r * kThreads < P ? exec_idx[p < P ? p : P - 1] : -1;
    }
}

// A workgroup barrier that leaves global loads in flight (__syncthreads would wait for the
// loads into LDS): this wavefront's LDS operations are done, then the others' are.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The pairs p < P with exec_idx[p] == e, in ascending order, into list[]; returns how
// many.  256 threads; P <= 1024 (four rounds of wave ballots).
__device__ int expert_pairs(const int (&ev)[kPairRounds], int P, int e, uint16_t *list,
                            int (*cnt)[4]) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    bool hit[kPairRounds];
    unsigned long long m[kPairRounds];
#pragma unroll
    for (int r = 0; r < kPairRounds; ++r) {
        hit[r] = r * kThreads + t < P && ev[r] == e;
        m[r] = __ballot(hit[r]);
        if (lane == 0) cnt[r][wave] = __popcll(m[r]);
    }
    lds_barrier();
    int base = 0;
#pragma unroll
    for (int r = 0; r < kPairRounds; ++r) {
        if (r * kThreads >= P) break;
        int off = base;
        for (int w = 0; w < wave; ++w) off += cnt[r][w];
        if (hit[r]) list[off + __popcll(m[r] & ((1ull << lane) - 1ull))] = uint16_t(r * kThreads + t);
        base += cnt[r][0] + cnt[r][1] + cnt[r][2] + cnt[r][3];
    }
    lds_barrier();
    return base;
}

// The K blocks of split z of a K range: units of plan_kb values (of which the split rule
// shares out whole ones, and in whose order the sums are formed whatever the size of a
// block), each of PER blocks of kb.  Units are visited from a rotated start: workgroups that
// run side by side then read different offsets of their rows instead of all hitting the
// same DRAM channels.  Blocks wholly past the end of K are left out.
template <int PER>
struct KBlocks {
    int lo, units, rot, kb;
    int nb;     // blocks of the split
    int gap;    // the first block behind those left out (the last unit's)
    int left;   // how many are left out
    __device__ __forceinline__ int k0(int b) const {
        if (PER > 1 && b >= gap) b += left;
        const int u = b / PER, q = u + rot;
        return ((lo + (q >= units ? q - units : q)) * PER + b % PER) * kb;
    }
};

template <int PER>
__device__ __forceinline__ KBlocks<PER> k_blocks(int K, int kb, int splits, int z) {
    const int n = (K + PER * kb - 1) / (PER * kb);
    KBlocks<PER> r;
    r.lo = z * n / splits;
    const int hi = (z + 1) * n / splits;
    r.units = hi - r.lo;
    r.kb = kb;
    r.rot = int((blockIdx.x * 7u + blockIdx.y * 13u) % unsigned(r.units > 0 ? r.units : 1));
    // the last unit of K is the split's last, visited units - 1 - rot units after the first
    r.left = hi == n && r.units > 0 ? (n * PER * kb - K) / kb : 0;
    r.gap = (r.units - r.rot) * PER - r.left;
    r.nb = r.units * PER - r.left;
    return r;
}

__device__ __forceinline__ uint4 widen8(WBf16, uint4 v, int, float) { return v; }
// 8 of a chunk's codes (the j-th eighth of 8) widened to bf16 exactly: E4M3 values are bf16
// values; an E2M1 value times its power-of-two scale too.
__device__ __forceinline__ uint4 widen8(WE4M3, uint4 v, int j, float) {
    const int c0 = int(j ? v.z : v.x), c1 = int(j ? v.w : v.y);
    const auto a = __builtin_amdgcn_cvt_pk_f32_fp8(c0, false);
    const auto b = __builtin_amdgcn_cvt_pk_f32_fp8(c0, true);
    const auto e = __builtin_amdgcn_cvt_pk_f32_fp8(c1, false);
    const auto f = __builtin_amdgcn_cvt_pk_f32_fp8(c1, true);
    const auto pk = [](float lo, float hi) {
        return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
    };
    return make_uint4(pk(a[0], a[1]), pk(b[0], b[1]), pk(e[0], e[1]), pk(f[0], f[1]));
}
__device__ __forceinline__ uint4 widen8(WMxfp4, uint4 v, int j, float sc) {
    const uint32_t c = j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
    return make_uint4(
        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, sc, 0)),
        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, sc, 1)),
        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, sc, 2)),
        __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(c, sc, 3)));
}

// Sizes of one workgroup's tile: NW matrices of 64 rows, up to 16 * MT tokens, K in blocks
// of KB values (one or two cache lines of every weight row).  Two weight stages are in LDS:
// one is multiplied while the other one loads.
// LDS decides how many workgroups share a CU, and more of them hide more than more stages
// do (the start of a workgroup: slot, pair scan, first activations; the last round of them).
// With three or four stages, for one projection, format and tile count at a time, calls ran
// at 0.93 to 1.01 of the speed with two.
// Two lines per row and block (W; a block is then the plan's unit) halve the barriers, for
// twice the LDS: see wide_rows.
// One activation buffer takes a barrier more per block, and pays where a CU then holds a
// workgroup more, up to four (32 tokens MXFP4 1.06 as a mean, 64 tokens E4M3 1.04, Granite-3B
// 16 tokens bf16 1.07).
// Calls of 221 shapes (2 to 64 tokens, six models with all or some experts resident, three
// formats) against the loop through registers with two barriers a block: 1.12 as a mean,
// 0.95 (DeepSeek-16B, 24 experts, 2 and 4 tokens MXFP4) to 1.57.
template <int NW, int MT, class WF, bool W>
struct TileShape {
    static constexpr int kRowBytes = W ? 256 : 128;   // of a weight row per block
    static constexpr int kChunks = kRowBytes / 16;
    static constexpr int KB = kChunks * WF::kChunkK;
    static constexpr int PER = WF::template plan_kb<MT>() / KB;   // blocks per unit of KBlocks
    static constexpr int kStage = NW * kRows * kRowBytes;
    static constexpr int kXRow = KB + 8;   // +16 B: the 16 rows of a fragment read hit distinct banks
    static constexpr int kXs = 16 * MT * kXRow * 2;
    static constexpr int kList = APEX_MAX_PAIRS * 2 + kPairRounds * 16 + 64;
    static constexpr int lds(int xb) { return 2 * kStage + xb * kXs + kList; }
    static constexpr int per_cu(int xb) { return std::min(160 * 1024 / lds(xb), 4); }
    static constexpr int XB = per_cu(1) > per_cu(2) ? 1 : 2;   // activation buffers
    static_assert(lds(XB) <= 80 * 1024 && WF::template plan_kb<MT>() % KB == 0, "tile");
};

template <int I>
struct Int {
    static constexpr int value = I;
};

// The permutation of a row's 16-byte chunks in LDS: the 16 rows of a fragment read, at the
// same chunk, then fall in distinct banks.
template <int RB>
__device__ __forceinline__ int swizzle(int row) {
    return RB == 256 ? row & 15 : row >> 1;
}

// The register's value is taken here: the compiler waits for the load that fills it at this
// point and moves no arithmetic on it to an earlier one.
__device__ __forceinline__ void settle(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void settle(ActF32::Raw &r) {
    asm volatile("" : "+v"(r.a.x), "+v"(r.a.y), "+v"(r.a.z), "+v"(r.a.w), "+v"(r.b.x), "+v"(r.b.y),
                      "+v"(r.b.z), "+v"(r.b.w));
}
__device__ __forceinline__ void settle(ActBf16::Raw &r) {
    asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));
}

// The s_waitcnt operand that waits until at most n (capped) vector loads are outstanding.
constexpr int vmcnt_only(int n) {
    n = n > 63 ? 63 : n;
    return 0x0f70 | (n & 15) | (n >> 4 << 14);
}

// The weights of block b (16 rows per wavefront and matrix) into a stage; a block past the
// last one loads nothing (offsets past the buffer's end).  Buffer loads: the compiler takes
// global loads into LDS for accesses of either memory and waits for all of them at the
// next use of any loaded register.
template <int NW, int RB, class WF, class KR>
__device__ __forceinline__ void load_weights(uint8_t *st, const uint8_t *const (&wbase)[NW],
                                             size_t wstride, int rows_valid, int K,
                                             const KR &kr, int b) {
    constexpr int CH = RB / 16, RPI = kWave / CH;   // chunks of a row, rows per instruction
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int k0 = kr.k0(min(b, kr.nb > 0 ? kr.nb - 1 : 0));
    const int row0 = min(16 * wave, rows_valid - 1);   // rows past the tile's last repeat it
    // In a scalar register by force: the select is made in a vector one, and a load whose
    // descriptor is not known to be uniform is wrapped in a loop over the lanes' values
    // (1172 of this file's 1822 direct loads, with the pipeline cut at each).
    const int bytes = __builtin_amdgcn_readfirstlane(b < kr.nb ? -1 : 0);
#pragma unroll
    for (int m = 0; m < NW; ++m) {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t *>(wbase[m]) + size_t(row0) * wstride, 0,
            uint32_t(bytes), 0x00027000);
#pragma unroll
        for (int i = 0; i < 16 / RPI; ++i) {
            const int row = RPI * i + lane / CH;             // of the wavefront's 16
            const int chunk = (lane % CH) ^ swizzle<RB>(row);
            const int k = min(k0 + chunk * WF::kChunkK, K - WF::kChunkK);
            const uint32_t at = uint32_t(min(row, rows_valid - 1 - row0)) * uint32_t(wstride) +
                                uint32_t(k) / WF::kChunkK * 16u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsrc,
                (__attribute__((address_space(3))) void *)(st + ((wave * NW + m) * 16 + RPI * i) * RB),
                16, at, 0, 0, 2 /* non-temporal */);
        }
    }
}

// Grouped-GEMM mainloop, shared by the gate/up and down projections and the weight
// formats.  A workgroup (4 wavefronts) owns a tile of 64 weight rows of NW weight
// matrices and up to 16 * NT tokens, over the K blocks of kr.
//
// Weights go from memory to LDS directly (16 bytes per lane, 8 rows of 128 bytes or 4 of 256
// per instruction), each wavefront loading the 16 rows that it multiplies: no barrier and no
// register stands between a weight load and its use, only the wavefront's own count of
// loads.  A row's chunks are permuted (by the lanes' addresses, the LDS side being linear)
// so that the 16 rows of a fragment read fall in distinct banks.  Codes stay codes in LDS
// and are widened to bf16 right before the matrix cores take them.  A lane multiplies the
// K values of its own chunks: the activations are read in the same order.
// Activations are the same for all four wavefronts: loaded a block ahead into registers,
// converted to bf16 and staged in LDS, with a barrier per block (two with one buffer).
// Loads return in order: a block's activations are requested before its weights, so that the
// wait for them leaves the weights in flight.
// Every load is unconditional (blocks past the last one read one cached line, rows past
// the last one that row) so that the compiler's load counts are exact.  K past the end is
// zero on both sides; rows and tokens past the end are multiplied and dropped.
template <int NW, int MT, int NT, bool W, class Act, class WF, class Stage>
__device__ __forceinline__ void gemm_tile(const Stage &stage, uint16_t *xs, bool w_ready,
                                          const uint8_t *const (&wbase)[NW], size_t wstride,
                                          const uint8_t *const (&sbase)[NW], size_t sstride,
                                          int rows_valid, int K,
                                          const KBlocks<TileShape<NW, MT, WF, W>::PER> &kr,
                                          const uint16_t *list, int n_tok, int list_div,
                                          const void *act, size_t act_stride,
                                          floatx4 (&acc)[NW][NT]) {
    using S = TileShape<NW, MT, WF, W>;
    constexpr int KB = S::KB;
    constexpr int SPR = KB / 8;                                    // 8-value pieces per token
    constexpr int XP = 16 * NT * SPR / kThreads > 0 ? 16 * NT * SPR / kThreads : 1;
    constexpr int P = S::kChunks / 4, SUB = WF::kChunkK / 8;          // matrix-core steps
    const int t = threadIdx.x, wave = t / kWave, lane = t % kWave;
    const int n = lane & 15, g = lane >> 4;
    // activation pieces of this thread (threads past the last piece repeat others')
    const uint8_t *xrow[XP];
    int xk[XP], xat[XP];
#pragma unroll
    for (int j = 0; j < XP; ++j) {
        const int p = (t + j * kThreads) % (16 * NT * SPR);
        const int row = p / SPR;
        xk[j] = 8 * (p % SPR);
        xat[j] = row * S::kXRow + xk[j];
        xrow[j] = static_cast<const uint8_t *>(act) +
                  list[row < n_tok ? row : 0] / list_div * act_stride;
    }
    // Loads that may still be on the way when block b is multiplied: those of the next one.
    // (The compiler does not tie a load into LDS to the reads of it.)
    constexpr int kInFlight =
        XP * Act::kLoads + (WF::kBlockScale ? NW * P : 0) + NW * S::kRowBytes / 64;
    typename Act::Raw x[XP];
    float sc[NW][P];
#pragma unroll
    for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[m][tt] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (kr.nb <= 0) return;
    const int row_c = min(16 * wave + n, rows_valid - 1);
    const auto load_x = [&](int b) {
        const int k0 = kr.k0(min(b, kr.nb - 1));
#pragma unroll
        for (int j = 0; j < XP; ++j) x[j] = Act::load(xrow[j], min(k0 + xk[j], K - 8));
        if constexpr (WF::kBlockScale)
#pragma unroll
            for (int m = 0; m < NW; ++m)
#pragma unroll
                for (int p = 0; p < P; ++p)
                    sc[m][p] = __uint_as_float(
                        sbase[m][size_t(row_c) * sstride + min(k0 / 32 + 4 * p + g, K / 32 - 1)]);
        __builtin_amdgcn_sched_barrier(0);
    };
    const auto settle_scales = [&] {
        if constexpr (WF::kBlockScale)
#pragma unroll
            for (int m = 0; m < NW; ++m)
#pragma unroll
                for (int p = 0; p < P; ++p) settle(sc[m][p]);
    };
    const auto block = [&](auto which, int b) {
        constexpr int I = decltype(which)::value;
        uint16_t *xb = xs + (S::XB == 2 ? I * (16 * MT * S::kXRow) : 0);
        const int end = b < kr.nb ? K : 0;   // a block past the last one multiplies zeros
        const int k0 = kr.k0(min(b, kr.nb - 1));
        if (S::XB == 1) lds_barrier();   // the previous block's activations have been read
#pragma unroll
        for (int j = 0; j < XP; ++j)
            *reinterpret_cast<uint4 *>(xb + xat[j]) = keep_if(Act::to_bf16(x[j]), k0 + xk[j] < end);
        settle_scales();
        float scale[NW][P];
#pragma unroll
        for (int m = 0; m < NW; ++m)
#pragma unroll
            for (int p = 0; p < P; ++p)
                scale[m][p] =
                    WF::kBlockScale ? apex::ffn::mx_scale(__float_as_uint(sc[m][p])) : 1.f;
        lds_barrier();
        load_x(b + 1);
        load_weights<NW, S::kRowBytes, WF>(stage(Int<1 - I>{}), wbase, wstride, rows_valid, K, kr, b + 1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_only(kInFlight));   // block b's weights are in LDS
        asm volatile("" ::: "memory");
        const uint8_t *w = stage(which) + wave * (NW * 16 * S::kRowBytes);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            uint4 raw[NW];
#pragma unroll
            for (int m = 0; m < NW; ++m)
                raw[m] = *reinterpret_cast<const uint4 *>(
                    w + (m * 16 + n) * S::kRowBytes + 16 * ((4 * p + g) ^ swizzle<S::kRowBytes>(n)));
#pragma unroll
            for (int m = 0; m < NW; ++m)
                raw[m] = keep_if(raw[m], k0 + (4 * p + g) * WF::kChunkK < end);
#pragma unroll
            for (int j = 0; j < SUB; ++j) {
                uint4 wop[NW];
#pragma unroll
                for (int m = 0; m < NW; ++m) wop[m] = widen8(WF{}, raw[m], j, scale[m][p]);
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    const uint4 xop = *reinterpret_cast<const uint4 *>(
                        xb + (16 * tt + n) * S::kXRow + 8 * ((4 * p + g) * SUB + j));
#pragma unroll
                    for (int m = 0; m < NW; ++m)
                        acc[m][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(xop), as_bf16x8(wop[m]), acc[m][tt], 0, 0, 0);
                }
            }
        }
        // the next block's wait for its activations stays behind these multiplies
        __builtin_amdgcn_sched_barrier(0);
    };
    load_x(0);
    if (!w_ready) load_weights<NW, S::kRowBytes, WF>(stage(Int<0>{}), wbase, wstride, rows_valid, K, kr, 0);
    // The first block's weights were requested before its activations where w_ready, after
    // them in the loop.  Both are needed at once: waiting for them here leaves one order of
    // requests at the top of the loop, where the compiler would otherwise wait for everything,
    // the next block's weights among it.
#pragma unroll
    for (int j = 0; j < XP; ++j) settle(x[j]);
    settle_scales();
    for (int b = 0; b < kr.nb; b += 2) {
        block(Int<0>{}, b);
        block(Int<1>{}, b + 1);
    }
    // no load into LDS may outlive its stage (the next pass or another workgroup's LDS)
    __builtin_amdgcn_s_waitcnt(0x0f70);
}

// The fp32 row scales of an apex_pack_expert_fp8 slot: W1 rows, W3 rows, W2 rows.
template <class WF>
__device__ __forceinline__ const float *row_scales(const typename WF::T *slot, int d, int I) {
    return reinterpret_cast<const float *>(slot + size_t(3) * I * d);
}

// The stages of a tile: LDS arrays of their own, so that the compiler tells a load into one
// from a read of another.
#define APEX_STAGES(NW_)                                                                       \
    using S = TileShape<NW_, MT, WF, W>;                                                       \
    __shared__ __align__(16) uint8_t st0[S::kStage], st1[S::kStage];                           \
    __shared__ __align__(16) uint16_t xs[S::XB * S::kXs / 2];                                  \
    __shared__ uint16_t list[APEX_MAX_PAIRS];                                                  \
    __shared__ int cnt[kPairRounds][4];                                                        \
    const auto stage = [&](auto i) -> uint8_t * { return decltype(i)::value == 0 ? st0 : st1; };

// up_gemm: grid (ceil(I / 64), E, SU).  64 rows of W1 and W3 of expert blockIdx.y, every
// token of the expert (16*MT per pass), K blocks of split blockIdx.z.  slot_stride is
// the slot size in elements of WF::T.
// SU == 1: hb[pair, i] = bf16(silu(W1[i] . x_b) * (W3[i] . x_b)), ungated.
// SU  > 1: uv[(2z) * P*I + pair*I + i] = W1[i] . x_b over the split, uv[(2z+1) ...] = W3.
// E4M3 slots: the dot products are multiplied by the rows' scales.
template <int MT, int SU, class WF, bool W>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void up_gemm(
    const float *__restrict__ x, int d, int I, int P, int k, const int32_t *__restrict__ exec_idx,
    const int32_t *__restrict__ slot_of_expert, int n_slots,
    const typename WF::T *__restrict__ slots, size_t slot_stride, __bf16 *__restrict__ hb,
    float *__restrict__ uv) {
    APEX_STAGES(2)
    const int e = blockIdx.y;
    int ev[kPairRounds];
    pair_ids(exec_idx, P, ev);
    const int s = slot_of_expert[e];
    if (s < 0 || s >= n_slots) return;
    const int i0 = blockIdx.x * kRows;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const typename WF::T *slot = slots + size_t(s) * slot_stride;
    const uint8_t *w1 = reinterpret_cast<const uint8_t *>(slot + size_t(i0) * 2 * d / WF::kKPerElem);
    const size_t row_bytes = size_t(d) / WF::kKPerElem * sizeof(typename WF::T);
    const uint8_t *const wbase[2] = {w1, w1 + row_bytes};
    const size_t wstride = 2 * row_bytes;
    // MXFP4 block scales of W1 and W3 rows i0.. (unused by the other formats)
    const uint8_t *sc = reinterpret_cast<const uint8_t *>(slot) + size_t(3) * I * d / 2;
    const uint8_t *const sbase[2] = {sc + size_t(i0) * (d / 32),
                                     sc + size_t(I + i0) * (d / 32)};
    const auto kr = k_blocks<S::PER>(d, S::KB, gridDim.z, blockIdx.z);
    // The first block's weights load while the expert's pairs are looked up.  An empty
    // split, or an expert without tokens, waits for them and drops them.
    load_weights<2, S::kRowBytes, WF>(st0, wbase, wstride, I - i0, d, kr, 0);
    const int n_e = expert_pairs(ev, P, e, list, cnt);
    const auto pass = [&](auto tiles, int t0) {
        constexpr int NT = decltype(tiles)::value;
        floatx4 acc[2][NT];
        gemm_tile<2, MT, NT, W, ActF32, WF>(stage, xs, t0 == 0, wbase, wstride, sbase, size_t(d / 32),
                                         I - i0, d, kr, list + t0, n_e - t0, k, x,
                                         size_t(d) * sizeof(float), acc);
        const int i = i0 + 16 * wave + (lane & 15);
        float s1 = 1.f, s3 = 1.f;
        if constexpr (WF::kFp8) {
            const float *sc = row_scales<WF>(slot, d, I);
            s1 = i < I ? sc[i] : 0.f;
            s3 = i < I ? sc[I + i] : 0.f;
        }
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int tok = t0 + 16 * tt + 4 * (lane >> 4) + r;
                if (tok < n_e && i < I) {
                    const size_t at = size_t(list[tok]) * I + i;
                    const float u = s1 * acc[0][tt][r], v = s3 * acc[1][tt][r];
                    if (SU == 1) {
                        hb[at] = (__bf16)(silu(u) * v);
                    } else {
                        uv[size_t(2 * blockIdx.z) * P * I + at] = u;
                        uv[size_t(2 * blockIdx.z + 1) * P * I + at] = v;
                    }
                }
            }
        __syncthreads();   // LDS is reused by the next pass
    };
    for (int t0 = 0; t0 < n_e; t0 += 16 * MT) {
        if (MT >= 2 && n_e - t0 <= 16) pass(Int<1>{}, t0);
        else if (MT >= 4 && n_e - t0 <= 32) pass(Int<2>{}, t0);
        else pass(Int<MT>{}, t0);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // no load into LDS outlives the workgroup
}

// down_gemm: grid (ceil(d / 64), E, SD).  64 rows j of W2 of expert blockIdx.y, K (= I)
// blocks of split blockIdx.z.  yp[z * P*d + pair*d + j] = W2[j] . h[pair] over the split.
// The activations are the bf16 h rows.
template <int MT, class WF, bool W>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void down_gemm(
    int d, int I, int P, const int32_t *__restrict__ exec_idx,
    const int32_t *__restrict__ slot_of_expert, int n_slots,
    const typename WF::T *__restrict__ slots, size_t slot_stride, const __bf16 *__restrict__ hb,
    float *__restrict__ yp) {
    APEX_STAGES(1)
    const int e = blockIdx.y;
    int ev[kPairRounds];
    pair_ids(exec_idx, P, ev);
    const int s = slot_of_expert[e];
    if (s < 0 || s >= n_slots) return;
    const int j0 = blockIdx.x * kRows;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const typename WF::T *slot = slots + size_t(s) * slot_stride;
    const uint8_t *const wbase[1] = {reinterpret_cast<const uint8_t *>(
        slot + (size_t(2) * I * d + size_t(j0) * I) / WF::kKPerElem)};
    const size_t wstride = size_t(I) / WF::kKPerElem * sizeof(typename WF::T);
    const uint8_t *const sbase[1] = {reinterpret_cast<const uint8_t *>(slot) +
                                     size_t(3) * I * d / 2 + size_t(2) * I * (d / 32) +
                                     size_t(j0) * (I / 32)};
    const auto kr = k_blocks<S::PER>(I, S::KB, gridDim.z, blockIdx.z);
    // the first block's weights load while the expert's pairs are looked up (as in up_gemm)
    load_weights<1, S::kRowBytes, WF>(st0, wbase, wstride, d - j0, I, kr, 0);
    const int n_e = expert_pairs(ev, P, e, list, cnt);
    float *out = yp + size_t(blockIdx.z) * P * d;
    const auto pass = [&](auto tiles, int t0) {
        constexpr int NT = decltype(tiles)::value;
        floatx4 acc[1][NT];
        gemm_tile<1, MT, NT, W, ActBf16, WF>(stage, xs, t0 == 0, wbase, wstride, sbase,
                                          size_t(I / 32), d - j0, I, kr, list + t0, n_e - t0, 1,
                                          hb, size_t(I) * sizeof(__bf16), acc);
        const int j = j0 + 16 * wave + (lane & 15);
        float s2 = 1.f;
        if constexpr (WF::kFp8) s2 = j < d ? row_scales<WF>(slot, d, I)[2 * I + j] : 0.f;
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int tok = t0 + 16 * tt + 4 * (lane >> 4) + r;
                if (tok < n_e && j < d)
                    out[size_t(list[tok]) * d + j] = s2 * acc[0][tt][r];
            }
        __syncthreads();   // LDS is reused by the next pass
    };
    for (int t0 = 0; t0 < n_e; t0 += 16 * MT) {
        if (MT >= 2 && n_e - t0 <= 16) pass(Int<1>{}, t0);
        else if (MT >= 4 && n_e - t0 <= 32) pass(Int<2>{}, t0);
        else pass(Int<MT>{}, t0);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // no load into LDS outlives the workgroup
}

// swiglu_reduce: h[pair, i] = bf16(silu(sum_z u_z) * sum_z v_z) from up_gemm's SU split
// partials (splits added in order), for the pairs whose expert has a slot; 8 consecutive
// i per thread.
template <int SU>
__global__ __launch_bounds__(kThreads) void swiglu_reduce(
    int P, int I, int E, const int32_t *__restrict__ exec_idx,
    const int32_t *__restrict__ slot_of_expert, int n_slots, const float *__restrict__ uv,
    __bf16 *__restrict__ hb) {
    const int per = I / 8;
    const int g = blockIdx.x * kThreads + threadIdx.x;
    if (g >= P * per) return;
    const int p = g / per, i = 8 * (g - p * per);
    const int e = exec_idx[p];
    if (e < 0 || e >= E) return;
    const int sl = slot_of_expert[e];
    if (sl < 0 || sl >= n_slots) return;
    const size_t at = size_t(p) * I + i;
    *reinterpret_cast<uint4 *>(hb + at) = swiglu8<SU>(uv + at, size_t(P) * I);
}

// combine: y[b, j] (+)= sum over positions q of token b, in position order, of
// gate[q] * (sum over splits z, in order, of yp[z, pair, j]) for the pairs this pass
// executed.  Four consecutive j per thread.  Lane q of every wavefront looks up position
// q (its expert, slot and gate; k <= 64 since k <= E), so all positions cost one chain of
// dependent loads, and the wavefront reads them back with readlane.  The partial outputs
// of a group of positions are loaded before any is added (those of positions that were
// not executed are read and dropped).
template <int SD>
__global__ __launch_bounds__(kThreads) void combine_pairs(
    int B, int d, int E, int k, const int32_t *__restrict__ exec_idx,
    const float *__restrict__ exec_gate, const int32_t *__restrict__ slot_of_expert, int n_slots,
    const float *__restrict__ yp, float *__restrict__ y, int accumulate) {
    constexpr int kGroup = SD <= 2 ? 8 : 4;
    const int b = blockIdx.y;
    const int j = 4 * (blockIdx.x * kThreads + threadIdx.x);
    const int lane = threadIdx.x % kWave;
    int pos_ok = 0;
    float pos_gate = 0.f;
    if (lane < k) {
        const int p = b * k + lane;
        const int e = exec_idx[p];
        const bool e_ok = e >= 0 && e < E;
        const int sl = slot_of_expert[e_ok ? e : 0];
        pos_ok = e_ok && sl >= 0 && sl < n_slots;
        pos_gate = exec_gate[p];
    }
    if (j >= d) return;
    const size_t Pd = size_t(B) * k * d;
    const float *row = yp + size_t(b) * k * d + j;
    float4 *dst = reinterpret_cast<float4 *>(y + size_t(b) * d + j);
    const float4 o = *dst;   // read whether or not it is added, so no branch waits on it
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const auto group = [&](int q0) {
        float4 v[kGroup][SD];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int q = min(q0 + u, k - 1);
#pragma unroll
            for (int z = 0; z < SD; ++z)
                v[u][z] = *reinterpret_cast<const float4 *>(row + z * Pd + size_t(q) * d);
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            if (q0 + u >= k) break;
            if (!__builtin_amdgcn_readlane(pos_ok, q0 + u)) continue;
            const float g = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pos_gate), q0 + u));
            float4 t = v[u][0];
#pragma unroll
            for (int z = 1; z < SD; ++z) {
                t.x += v[u][z].x; t.y += v[u][z].y; t.z += v[u][z].z; t.w += v[u][z].w;
            }
            s.x += g * t.x; s.y += g * t.y; s.z += g * t.z; s.w += g * t.w;
        }
    };
    group(0);   // outside the loop, so its loads issue together with the read of y
    for (int q0 = kGroup; q0 < k; q0 += kGroup) group(q0);
    if (accumulate) s = make_float4(o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w);
    *dst = s;
}

// K splits of a projection with `groups` workgroups of work (row tiles times experts)
// and `nb` K blocks: `target` workgroups over all splits (rounded to the nearest split
// count when `nearest`, else up), at most kMaxSplit, and at least `min_blocks` K blocks
// per split.
int pick_splits(int groups, int nb, int target, bool nearest, int min_blocks) {
    groups = std::max(1, groups);
    int s = nearest ? (target + groups / 2) / groups : (target + groups - 1) / groups;
    s = std::min(s, kMaxSplit);
    s = std::min(s, std::max(1, nb / min_blocks));
    return std::max(s, 1);
}

struct Plan {
    int MT, SU, SD;
    size_t uv_bytes, h_bytes, y_bytes;   // h_bytes: the split partials (if any) and h
};

// The launch plan for weight format WF.  The split rules were fitted to timings of
// every split pair (1-4 each) on grouped calls of the Granite-3B, OLMoE, Mixtral,
// DeepSeek-16B and Phi-7B expert shapes in all three formats (24 to 64 resident
// experts), on an earlier loop that took the weights through registers; they have not been
// fitted again, so that the order of the sums stays as it was.  Each K split adds a
// prologue (finding the expert's pairs, the first load) and partial sums, and pays only
// when the projection has too few workgroups to keep HBM busy.  The gate/up target grows
// with the per-byte cost of widening the codes (bf16 none, E4M3 most per byte); the down
// projection splits only over long K (for Mixtral's I = 14336).  On that loop the rule was
// within 1 % of the best split pair on average over those calls.
template <class WF>
Plan plan_for(int B, int d, int I, int k, int E, int n_slots) {
    Plan pl;
    // token tiles per pass: enough for the whole batch on one expert up to 64 tokens
    pl.MT = B >= 48 ? 4 : (B >= 24 ? 2 : 1);
    const int experts = std::min(std::min(E, B * k), n_slots);
    const int kb = pl.MT == 4   ? WF::template plan_kb<4>()
                   : pl.MT == 2 ? WF::template plan_kb<2>()
                                : WF::template plan_kb<1>();
    const int nb_d = (d + kb - 1) / kb, nb_i = (I + kb - 1) / kb;
    pl.SU = pick_splits((I + kRows - 1) / kRows * experts, nb_d, WF::kUpGroups, true, 3);
    pl.SD = pick_splits((d + kRows - 1) / kRows * experts, nb_i, 1024, false, 8);
    const size_t P = size_t(B) * k;
    pl.uv_bytes =
        pl.SU == 1 ? 0 : apex::align_up(size_t(2) * pl.SU * P * I * sizeof(float), 256);
    pl.h_bytes = pl.uv_bytes + P * I * 2;
    pl.y_bytes = size_t(pl.SD) * P * d * sizeof(float);
    return pl;
}

// LDS to ask for beyond a tile's own, so that a CU takes at most an even share of the launch:
// the hardware fills a CU before it looks at the next one, and while it does, the workgroups of
// experts without a slot come and go, so that some CUs end up with three or four workgroups
// and others with none.  The number per CU (two at least) is the one with which the rounds of
// workgroups (of up to 1024; more level out by themselves) take least, a round's time going
// by how many share the CU.  Counted are the experts that have a slot: those without tokens
// load a block and leave, and would hold up the others.
// us a call, without -> with: OLMoE, 24 experts of 64 resident, 64 tokens bf16 77.8 -> 65.4 (three
// stages, so two workgroups a CU: 68.2), all resident 142.8 -> 130.0; Mixtral 4 of 8, 32 tokens
// E4M3 143.5 -> 132.8; OLMoE 24, 8 tokens MXFP4 36.6 -> 29.8.  Over 221 shapes 1.02 as a mean,
// 0.92 (OLMoE 24, 16 tokens E4M3) to 1.23.
template <class S>
size_t lds_pad(dim3 g, int experts) {
    const int n = int(g.x * g.z) * experts, most = std::min(160 * 1024 / S::lds(S::XB), 8);
    if (n > 1024) return 0;
    int per = most, best = INT_MAX;
    for (int c = most; c >= 2; --c) {
        const int time = (n + 256 * c - 1) / (256 * c) * c;
        if (time < best) best = time, per = c;
    }
    return per == most ? 0 : std::max(0, 160 * 1024 / (per + 1) + 1024 - S::lds(S::XB));
}

// Which of one and two lines per row (W) a projection, tile count and format has kernels for.
template <int NW, int MT, class WF, bool W>
constexpr bool has_rows() {
    if (WF::kChunkK == 16 && MT == 1) return true;
    return W == (WF::kChunkK == 8 && (NW == 1 || MT <= 2));
}

// Whether a launch with K splits of `units` units takes blocks of two lines per row.  bf16:
// always but for gate/up of 48 tokens and more, where two stages of them would leave no room
// for a second workgroup (with one line the speed is: down up to 23 tokens 0.91, 24 to 47 0.93,
// 48 and more 0.94, gate/up 0.93).  MXFP4: never (down up to 23 tokens with two: 1.01 over drawn
// shapes, but 0.95 at those of six models).  E4M3: up to
// 23 tokens (more have one line as their unit), unless a split is short and the launch large,
// where the workgroups that two lines leave no room for count for more: Granite-3B, 16 tokens,
// all 40 experts 35.6 us a call with two lines, 28.7 with one, but Mixtral, 4 tokens, 121 and
// 136, 64 experts of 3952 x 1808, 10 tokens, 153 and 188.  Figures: means over shapes drawn from 256
// to 4096 x 14336 with 4 to 64 experts.
template <int NW, int MT, class WF>
bool wide_rows(dim3 g, int experts, int units) {
    if (!has_rows<NW, MT, WF, true>()) return false;
    if (!has_rows<NW, MT, WF, false>()) return true;
    return units > 4 || int(g.x * g.z) * experts <= 512;
}
template <int MT, int SU, class WF, bool W, class... A>
void launch_up(dim3 g, int experts, hipStream_t st, A... a) {
    if constexpr (has_rows<2, MT, WF, W>())
        hipLaunchKernelGGL((up_gemm<MT, SU, WF, W>), g, dim3(kThreads),
                           (lds_pad<TileShape<2, MT, WF, W>>(g, experts)), st, a...);
}

template <int MT, class WF, bool W, class... A>
void launch_up_splits(dim3 g, int experts, hipStream_t st, A... a) {
    if (g.z == 1)
        launch_up<MT, 1, WF, W>(g, experts, st, a...);
    else if (g.z == 2)
        launch_up<MT, 2, WF, W>(g, experts, st, a...);
    else if (g.z == 3)
        launch_up<MT, 3, WF, W>(g, experts, st, a...);
    else
        launch_up<MT, 4, WF, W>(g, experts, st, a...);
}

template <int MT, class WF, bool W, class... A>
void launch_down(dim3 g, int experts, hipStream_t st, A... a) {
    if constexpr (has_rows<1, MT, WF, W>())
        hipLaunchKernelGGL((down_gemm<MT, WF, W>), g, dim3(kThreads),
                           (lds_pad<TileShape<1, MT, WF, W>>(g, experts)), st, a...);
}

// The gate/up and the down launch for MT token tiles per pass.
template <int MT, class WF, class... A>
void run_up(dim3 g, int experts, int K, hipStream_t st, A... a) {
    const int unit = WF::template plan_kb<MT>() * int(g.z), units = (K + unit - 1) / unit;
    if (wide_rows<2, MT, WF>(g, experts, units))
        launch_up_splits<MT, WF, true>(g, experts, st, a...);
    else
        launch_up_splits<MT, WF, false>(g, experts, st, a...);
}
template <int MT, class WF, class... A>
void run_down(dim3 g, int experts, int K, hipStream_t st, A... a) {
    const int unit = WF::template plan_kb<MT>() * int(g.z), units = (K + unit - 1) / unit;
    if (wide_rows<1, MT, WF>(g, experts, units))
        launch_down<MT, WF, true>(g, experts, st, a...);
    else
        launch_down<MT, WF, false>(g, experts, st, a...);
}

// The launches of one call for slots of weight format WF.
template <class WF>
apex_status run_grouped(const float *x, int B, int d, int I, int E, int k,
                        const int32_t *exec_idx, const float *exec_gate,
                        const int32_t *soe, const typename WF::T *slots, size_t stride,
                        int n_slots, float *y, int accumulate, char *wsb, hipStream_t stream) {
    const Plan pl = plan_for<WF>(B, d, I, k, E, n_slots);
    const int P = B * k;
    const int experts = std::min(E, n_slots);
    float *uv = reinterpret_cast<float *>(wsb);
    __bf16 *hb = reinterpret_cast<__bf16 *>(wsb + pl.uv_bytes);
    float *yp = reinterpret_cast<float *>(wsb + apex::align_up(pl.h_bytes, 256));
    const dim3 gu((I + kRows - 1) / kRows, E, pl.SU);
    if (pl.MT == 4)
        run_up<4, WF>(gu, experts, d, stream, x, d, I, P, k, exec_idx, soe, n_slots, slots, stride, hb, uv);
    else if (pl.MT == 2)
        run_up<2, WF>(gu, experts, d, stream, x, d, I, P, k, exec_idx, soe, n_slots, slots, stride, hb, uv);
    else
        run_up<1, WF>(gu, experts, d, stream, x, d, I, P, k, exec_idx, soe, n_slots, slots, stride, hb, uv);
    APEX_HIP(hipGetLastError());
    if (pl.SU > 1) {
        const dim3 gr((P * (I / 8) + kThreads - 1) / kThreads);
        if (pl.SU == 2)
            hipLaunchKernelGGL(swiglu_reduce<2>, gr, dim3(kThreads), 0, stream, P, I, E, exec_idx,
                               soe, n_slots, uv, hb);
        else if (pl.SU == 3)
            hipLaunchKernelGGL(swiglu_reduce<3>, gr, dim3(kThreads), 0, stream, P, I, E, exec_idx,
                               soe, n_slots, uv, hb);
        else
            hipLaunchKernelGGL(swiglu_reduce<4>, gr, dim3(kThreads), 0, stream, P, I, E, exec_idx,
                               soe, n_slots, uv, hb);
        APEX_HIP(hipGetLastError());
    }

    const dim3 gd((d + kRows - 1) / kRows, E, pl.SD);
    const __bf16 *hbc = hb;
    if (pl.MT == 4)
        run_down<4, WF>(gd, experts, I, stream, d, I, P, exec_idx, soe, n_slots, slots, stride, hbc, yp);
    else if (pl.MT == 2)
        run_down<2, WF>(gd, experts, I, stream, d, I, P, exec_idx, soe, n_slots, slots, stride, hbc, yp);
    else
        run_down<1, WF>(gd, experts, I, stream, d, I, P, exec_idx, soe, n_slots, slots, stride, hbc, yp);
    APEX_HIP(hipGetLastError());
    const dim3 gc((d / 4 + kThreads - 1) / kThreads, B);
    if (pl.SD == 1)
        hipLaunchKernelGGL(combine_pairs<1>, gc, dim3(kThreads), 0, stream, B, d, E, k, exec_idx,
                           exec_gate, soe, n_slots, yp, y, accumulate);
    else if (pl.SD == 2)
        hipLaunchKernelGGL(combine_pairs<2>, gc, dim3(kThreads), 0, stream, B, d, E, k, exec_idx,
                           exec_gate, soe, n_slots, yp, y, accumulate);
    else if (pl.SD == 3)
        hipLaunchKernelGGL(combine_pairs<3>, gc, dim3(kThreads), 0, stream, B, d, E, k, exec_idx,
                           exec_gate, soe, n_slots, yp, y, accumulate);
    else
        hipLaunchKernelGGL(combine_pairs<4>, gc, dim3(kThreads), 0, stream, B, d, E, k, exec_idx,
                           exec_gate, soe, n_slots, yp, y, accumulate);
    APEX_HIP(hipGetLastError());
    return APEX_OK;
}

}  // namespace

namespace apex {

// [2*SU fp32 split partials, when SU > 1][h: bf16 B*k x I][per-split, per-pair outputs:
//  SD x B*k x d fp32]
size_t ffn_grouped_workspace(int B, int d, int I, int k) {
    // the largest plan over the slot counts and weight formats the call can be given
    size_t worst = 0;
    const auto cover = [&](const Plan &pl) {
        worst = std::max(worst, align_up(pl.h_bytes, 256) + align_up(pl.y_bytes, 256));
    };
    for (int experts = 1; experts <= APEX_MAX_EXPERTS; ++experts) {
        cover(plan_for<WBf16>(B, d, I, k, APEX_MAX_EXPERTS, experts));
        cover(plan_for<WE4M3>(B, d, I, k, APEX_MAX_EXPERTS, experts));
        cover(plan_for<WMxfp4>(B, d, I, k, APEX_MAX_EXPERTS, experts));
    }
    return worst;
}

void ffn_grouped_plan(int B, int d, int I, int E, int k, int n_slots, WeightFormat fmt,
                      int32_t out[3]) {
    const Plan pl = fmt == WeightFormat::kE4M3    ? plan_for<WE4M3>(B, d, I, k, E, n_slots)
                    : fmt == WeightFormat::kMxfp4 ? plan_for<WMxfp4>(B, d, I, k, E, n_slots)
                                                  : plan_for<WBf16>(B, d, I, k, E, n_slots);
    out[0] = pl.MT;
    out[1] = pl.SU;
    out[2] = pl.SD;
}

apex_status ffn_grouped(const float *x, int B, int d, int I, int E, int k,
                        const int32_t *exec_idx, const float *exec_gate,
                        const int32_t *slot_of_expert, const void *slots, int n_slots,
                        WeightFormat fmt, float *y, int accumulate, void *workspace,
                        hipStream_t stream) {
    char *wsb = static_cast<char *>(workspace);
    if (fmt == WeightFormat::kE4M3)
        return run_grouped<WE4M3>(x, B, d, I, E, k, exec_idx, exec_gate, slot_of_expert,
                                  static_cast<const uint8_t *>(slots),
                                  apex_expert_bytes_fp8(d, I), n_slots, y, accumulate, wsb,
                                  stream);
    if (fmt == WeightFormat::kMxfp4)
        return run_grouped<WMxfp4>(x, B, d, I, E, k, exec_idx, exec_gate, slot_of_expert,
                                   static_cast<const uint8_t *>(slots),
                                   apex_expert_bytes_mxfp4(d, I), n_slots, y, accumulate, wsb,
                                   stream);
    return run_grouped<WBf16>(x, B, d, I, E, k, exec_idx, exec_gate, slot_of_expert,
                              static_cast<const uint16_t *>(slots), size_t(3) * d * I, n_slots,
                              y, accumulate, wsb, stream);
}

}  // namespace apex
