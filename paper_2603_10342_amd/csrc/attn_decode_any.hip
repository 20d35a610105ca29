// Decode over paged KV caches of any supported head_dim and dtype with pages of 16 tokens or more (bf16 with
// head_dim 128 on 16-token pages has a kernel of its own, attn_decode_mfma.hip).
//
// Bound by HBM, like that kernel, and built like it: the batch's (session, KV head) contexts are laid end to end in
// steps of 32 tokens and dealt to the workgroups in equal shares (find_share), all query heads of a KV head share
// one pass over the keys and values, both contractions run on the matrix cores with the heads padded to 16 columns,
// and a merge kernel combines the segments' partials in order.  Groups of more than 16 heads are cut into blocks
// of 16, each a pair of its own.  What differs:
//   - Arithmetic keeps 32 bits where the caches do: fp32 runs on 16x16x4 fp32 products, with up to four heads on 4x4x1 ones
//     (attend_few), with expf on unscaled exponents; bf16 caches
//     multiply the weights as three bf16 terms (bf16_terms.h), so that they stay in 32 bits.
//   - The 16-token group is the unit of addressing: group i of a context lies in page i / (page_size / 16), and a
//     group's keys and values sit in the page as in a 16-token page, only with a larger chunk stride for K.
//   - Two sub-steps of loads are in flight per wave where a sub-step is 16 KiB or less (head_dim 64 and 128):
//     with half the bytes per token, one in flight does not cover the latency.
//   - At 256 channels a sub-step's operands and O^T fill the registers: the fp32 split kernel spills 13, outside its step
//     loop; the dimensions between 128 and 256, which run as 256 with bounds, spill 45 (bf16: 26), 13 (5) of them read back
//     in every step.
// Whole decode step, append included (one wave per (row, query head) before -> now): 16 fp32 sessions of 1024..4096
// tokens at 32 / 8 heads x 128, 2760 -> 75 us (369 MB; 65.1 since up to four heads have products of their own, 5.7 TB/s); 48 bf16 sessions of 700..5000 at
// head_dim 64, 32-token pages, 2238 -> 63.5 us (333 MB, 5.2 TB/s; 62.8 with weights in two terms); two fp32 sessions of 300, 4 / 2 heads x 64, 106 -> 12 us.
// head_dim below its template's DT: loads beyond head_dim repeat its last channels; keys become zeros (as the query
// does), values land in rows that are not stored.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "attn_general_row.h"
#include "attn_split_common.h"
#include "bf16_terms.h"

namespace ag {

namespace {

using splitk::f32x4;
using splitk::u32x4;
using splitk::bf16x8;
using splitk::kLog2e;
using splitk::steps_of;

constexpr int kCols = 16;               // query heads of a pair (a block of the group's heads)

template <typename E>
__device__ __forceinline__ u32x4 load16(const E* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));    // read once per step
}

template <typename E, int DT>
struct SubStep {
    static constexpr bool kBf16 = sizeof(E) == 2;
    static constexpr int kTok = kBf16 ? 32 : 16;                 // tokens
    static constexpr int kK = kBf16 ? DT / 16 : DT / 16;         // 16-byte loads of a lane: keys
    static constexpr int kV = DT / 16;                           // ... and values
    u32x4 k[kK], v[kV];
};

template <typename E, int DT>
constexpr int q_row() { return DT * (int)sizeof(E) + 16; }      // bytes of a query row in LDS, padded

// The queries of a pair (heads h0 .. h0 + nh - 1 of a group) into LDS, rows padded and zero behind the last head and channel.
template <typename E, int DT, bool kExact, int kThreads>
__device__ __forceinline__ void queries_to_lds(const AttnArgs& a, int s, int g, int h0, int nh, unsigned char* s_q)
{
    constexpr int kPieces = DT * (int)sizeof(E) / 16;            // of a query row
    const int D = kExact ? DT : a.c.d, pieces = D * (int)sizeof(E) / 16, G = a.hq / a.c.hkv;
    const unsigned char* qs = (const unsigned char*)a.q + ((int64_t)s * a.hq + (int64_t)g * G + h0) * D * (int)sizeof(E);
    for (int idx = threadIdx.x; idx < kCols * kPieces; idx += kThreads) {
        const int head = idx / kPieces, p = idx - head * kPieces;
        u32x4 x = {0, 0, 0, 0};
        if (head < nh && p < pieces) x = *reinterpret_cast<const u32x4*>(qs + ((int64_t)head * pieces + p) * 16);
        *reinterpret_cast<u32x4*>(s_q + head * q_row<E, DT>() + p * 16) = x;
    }
}

// One wave's part of a pair's keys - sub-steps first, first + kStride, ... , `subs` of them - of (session s, KV head g, heads h0 ..
// h0 + nh - 1 of its group), whose context has ctx tokens: running maximum, sum and O^T of the heads.  my_pid: lane i holds
// the page of the i-th 16-token group of these sub-steps (of a group behind the last one, anything).  Contains one workgroup barrier
// (the queries are in LDS behind it).
template <typename E, int DT, bool kExact, int kStride>
__device__ __forceinline__ void attend_steps(const AttnArgs& a, int g, int ctx, int first, int subs, int my_pid,
                                             const unsigned char* s_q, float& m, float& lsum, f32x4 (&o)[DT / 16])
{
    using X = SubStep<E, DT>;
    constexpr bool kBf16 = X::kBf16;
    constexpr bool kTwoInFlight = X::kK + X::kV <= 16;
    constexpr int kQRow = q_row<E, DT>();
    const int hkv = a.c.hkv;
    const int D = kExact ? DT : a.c.d, ps = a.c.ps;
    const int lane = threadIdx.x & 63;

    const int r = lane & 15, c = lane >> 4;
    const int gmask = (1 << (a.c.ps_shift - 4)) - 1;            // 16-token groups of a page
    const int64_t block = (int64_t)D * ps;                       // elements of one (page, head)
    // bf16: score row r is slot r & 7 of group r >> 3, the second product takes slots 8..15, so that lane group c owns
    // the 8 tokens of value chunk c & 1 of group c >> 1.  fp32: score row r is slot r, lane group c owns tokens
    // 4 c .. 4 c + 3: elements 4 (c >> 1) .. + 3 of value chunk c & 1.
    const int k_slot = kBf16 ? (r & 7) * 8 : r * 8 + (c & 1) * 4;
    const int k_chunk = kBf16 ? c : c >> 1;                      // + 4 (bf16) or 2 (fp32) per load
    const int v_lane = kBf16 ? ((c & 1) * D) * 8 : ((c & 1) * D) * 8 + (c >> 1) * 4;
    const float unit = kBf16 ? a.scale * kLog2e : a.scale;       // bf16 takes its weights as powers of two
    auto power = [](float x) { return kBf16 ? __builtin_amdgcn_exp2f(x) : expf(x); };

    const int last_grp = (ctx - 1) >> 4;
    const E* kpool = (const E*)a.c.k;
    const E* vpool = (const E*)a.c.v;
    auto load = [&](X& x, int i) {                           // sub-step i of the wave
        if constexpr (kBf16) {
            const int grp = 2 * (first + kStride * i);       // (the second group may lie behind the last one)
            const int64_t pA = __builtin_amdgcn_readlane(my_pid, 2 * i), pB = grp < last_grp ? __builtin_amdgcn_readlane(my_pid, 2 * i + 1) : pA;
            const int gA = grp & gmask, gB = min(grp + 1, last_grp) & gmask;
            const int64_t baseA = (pA * hkv + g) * block, baseB = (pB * hkv + g) * block;
            const E* kp = kpool + (r >> 3 ? baseB + gB * 128 : baseA + gA * 128) + k_slot;
            const E* vp = vpool + (c >> 1 ? baseB + gB * 16 * D : baseA + gA * 16 * D) + v_lane;
#pragma unroll
            for (int kk = 0; kk < X::kK / 2; ++kk) {
                const int chunk = kExact ? k_chunk + 4 * kk : min(k_chunk + 4 * kk, (D >> 3) - 1);
                x.k[2 * kk] = load16(kp + (int64_t)chunk * ps * 8);
                x.k[2 * kk + 1] = load16(kp + (int64_t)chunk * ps * 8 + 64);
                if (!kExact && chunk != k_chunk + 4 * kk) x.k[2 * kk] = x.k[2 * kk + 1] = u32x4{0, 0, 0, 0};
            }
#pragma unroll
            for (int mb = 0; mb < X::kV; ++mb) x.v[mb] = load16(vp + (kExact ? mb * 16 + r : min(mb * 16 + r, D - 1)) * 8);
        } else {
            const int64_t p = __builtin_amdgcn_readlane(my_pid, i);
            const int gi = min(first + kStride * i, last_grp) & gmask;
            const int64_t at = (p * hkv + g) * block;
            const E* kp = kpool + at + gi * 128 + k_slot;
            const E* vp = vpool + at + gi * 16 * D + v_lane;
#pragma unroll
            for (int kk = 0; kk < X::kK; ++kk) {
                const int chunk = kExact ? k_chunk + 2 * kk : min(k_chunk + 2 * kk, (D >> 3) - 1);
                x.k[kk] = load16(kp + (int64_t)chunk * ps * 8);
                if (!kExact && chunk != k_chunk + 2 * kk) x.k[kk] = u32x4{0, 0, 0, 0};
            }
#pragma unroll
            for (int mb = 0; mb < X::kV; ++mb) x.v[mb] = load16(vp + (kExact ? mb * 16 + r : min(mb * 16 + r, D - 1)) * 8);
        }
    };

    m = -INFINITY;
    lsum = 0.0f;
#pragma unroll
    for (int mb = 0; mb < DT / 16; ++mb) o[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* q_lane = s_q + r * kQRow + c * 16;

    auto compute = [&](X& x, int i) {
        constexpr int kScores = kBf16 ? 8 : 4;
        const int tok0 = (first + kStride * i) * X::kTok;
        const int tokb = kBf16 ? tok0 + (c >> 1) * 16 + (c & 1) * 4 : tok0 + c * 4;
        const int keep = ctx - tokb;                         // token tokb + j exists iff j < keep
        f32x4 s1 = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
        float xs[kScores];
        if constexpr (kBf16) {
#pragma unroll
            for (int kk = 0; kk < X::kK / 2; ++kk) {
                const bf16x8 qk = *reinterpret_cast<const bf16x8*>(q_lane + kk * 64);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x.k[2 * kk]), qk, s1, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x.k[2 * kk + 1]), qk, s2, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                xs[j] = j < keep ? s1[j] * unit : -INFINITY;
                xs[4 + j] = 8 + j < keep ? s2[j] * unit : -INFINITY;
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < X::kK; ++kk) {
                const f32x4 qk = *reinterpret_cast<const f32x4*>(q_lane + kk * 64);
                const f32x4 kv = __builtin_bit_cast(f32x4, x.k[kk]);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[0], qk[0], s1, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[1], qk[1], s2, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[2], qk[2], s1, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[3], qk[3], s2, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) xs[j] = j < keep ? (s1[j] + s2[j]) * unit : -INFINITY;
        }
        float mx = fmaxf(fmaxf(xs[0], xs[1]), fmaxf(xs[2], xs[3]));
        if constexpr (kBf16) mx = fmaxf(mx, fmaxf(fmaxf(xs[4], xs[5]), fmaxf(xs[6], xs[7])));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        // (fp32: the second sub-step of a context's last step may hold no token)
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = power(m - m_ref);
        float p[kScores], psum = 0.f;
#pragma unroll
        for (int j = 0; j < kScores; ++j) { p[j] = power(xs[j] - m_ref); psum += p[j]; }
        lsum = lsum * alpha + psum;
        m = m_new;
        if (tok0 + X::kTok > ctx) {          // slots past the last token may hold anything, NaN included
#pragma unroll
            for (int mb = 0; mb < X::kV; ++mb) {
                if constexpr (kBf16) {
                    x.v[mb] = __builtin_bit_cast(u32x4, splitk::keep_quads(__builtin_bit_cast(bf16x8, x.v[mb]), keep, keep - 8));
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x.v[mb][j] = j < keep ? x.v[mb][j] : 0u;
                }
            }
        }
        if constexpr (kBf16) {
            Terms w;
#pragma unroll
            for (int j = 0; j < 4; ++j) w.set_pair(j, p[2 * j], p[2 * j + 1]);
#pragma unroll
            for (int mb = 0; mb < X::kV; ++mb) {
                const bf16x8 v = __builtin_bit_cast(bf16x8, x.v[mb]);
                o[mb] *= alpha;
                o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, __builtin_bit_cast(bf16x8, w.l), o[mb], 0, 0, 0);
                o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, __builtin_bit_cast(bf16x8, w.m), o[mb], 0, 0, 0);
                o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, __builtin_bit_cast(bf16x8, w.h), o[mb], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int mb = 0; mb < X::kV; ++mb) o[mb] *= alpha;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mb = 0; mb < X::kV; ++mb)
                    o[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4, x.v[mb])[j], p[j], o[mb], 0, 0, 0);
        }
    };

    if constexpr (kTwoInFlight) {
        X x0, x1;
        if (subs > 0) load(x0, 0);
        __syncthreads();                                     // Q is in LDS
#pragma unroll 1
        for (int i = 0; i < subs; i += 2) {
            if (i + 1 < subs) load(x1, i + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(x0, i);
            if (i + 2 < subs) load(x0, i + 2);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < subs) compute(x1, i + 1);
        }
    } else {
        X x;
        __syncthreads();
#pragma unroll 1
        for (int i = 0; i < subs; ++i) {
            load(x, i);
            __builtin_amdgcn_sched_barrier(0);               // all loads in flight before anything waits
            compute(x, i);
        }
    }
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
}

// ---- fp32, at most four query heads a pair, head_dim DT = 64 or 128 --------------------------------------------
// The 16 columns of the 16x16x4 products are mostly padding there, and they are what a short step waits for (two sessions of 300
// tokens at 4 / 2 heads x 64: 2.3 us of a step's 7 for the second and third sub-step of a wave).  The 4x4x1 products have four
// columns: 16 independent blocks of 4 x 4, at the same rate a product.  A sub-step of a wave is 32 tokens; lane = 32 u + l:
//   scores  rows = heads, columns = tokens.  B: keys, a lane holds four of eight channels of a token (the 32 bytes that a token has in
//           a chunk lie in lanes l and l + 32 of one load); A: the queries' two channels, each broadcast to its half of the blocks
//           from the one that holds it.  The halves' sums are added, so that both hold all 32 tokens.
//   a 4 x 4 transpose inside each quad of lanes turns "lane = token, register = head" into "lane = head, register = token"
//   values  rows = heads, columns = channels.  B: values, a lane holds four of the eight tokens of a chunk (slots below 8 in the lower
//           lanes, the others in the upper: one load is 1 KiB without gaps); A: the weights of the two tokens, each broadcast
//           to its half.  (Loads of every other 16 bytes, two for the same lines, cost up to 20 % of a batch that HBM bounds.)
// Neighbouring products write different accumulators, and every sum is shorter than with the other products.
// Graph replay, append included, 16x16x4 -> 4x4x1, us: 16 sessions of 1024..4096 at 32 / 8 x 128 72.1 -> 65.1 (369 MB), 8 of 100..500 27.1
// -> 18.0, one of 800 21.3 -> 14.8; at 64 channels one of 300 at 4 / 2 9.2 -> 7.2, 48 of 1000..4000 at 32 / 8 86.5 -> 82.6, of 60..110 10.3 ->
// 8.9; a session of two at 4 / 2 x 64 with 16 decode steps 171 -> 139.5.  97 batches 1.05 to 1.5 times faster.  Sub-steps of 64 tokens at
// 64 channels: 0.89 to 1.4.
constexpr int kFewHeads = 4;

template <int kCtrl>
__device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xF, 0xF, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowRor4 = 0x124, kRowRor8 = 0x128;
struct Two { float x, y; };
// {x of the lower half, y of the lower half} and {x of the upper, y of the upper} ...
__device__ __forceinline__ Two swap_halves(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return Two{__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
}
// ... the same of even and odd rows of 16 lanes
__device__ __forceinline__ Two swap_rows(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    return Two{__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])};
}
// x[i] of lane 4 b + j becomes x[j] of lane 4 b + i
__device__ __forceinline__ void transpose_quads(f32x4& x, int lane)
{
    const bool odd = lane & 1, upper = lane & 2;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const float got = dpp<kQuadXor1>(odd ? x[i] : x[i + 1]);
        if (odd) x[i] = got; else x[i + 1] = got;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float got = dpp<kQuadXor2>(upper ? x[i] : x[i + 2]);
        if (upper) x[i] = got; else x[i + 2] = got;
    }
}
template <class F, int... I>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }

constexpr int kFewTokens = 32;                                   // of a sub-step

// One wave's part of a pair: sub-steps of tokens token0 + i * kStep, `subs` of them, tokens below `end` only (at most the context's
// length).  my_pid: lane kGroups * i + k holds the page of group k of sub-step i (of a group behind the last one, anything).
// m, lsum: of head lane & 3, in every lane; o[h][i]: O of head i at channel 64 h + lane.
template <int DT, int kStep>
__device__ __forceinline__ void attend_few(const AttnArgs& a, int s, int g, int nh, int ctx, int end, int token0, int subs, int my_pid,
                                           float& m, float& lsum, f32x4 (&o)[DT / 64])
{
    constexpr int kTok = kFewTokens, kGroups = kTok / 16, kBlocks = DT / 32;         // kBlocks of 32 channels
    const int hkv = a.c.hkv, ps = a.c.ps, lane = threadIdx.x & 63, l = lane & 31, u = lane >> 5;
    const int gmask = (1 << (a.c.ps_shift - 4)) - 1, last_grp = (ctx - 1) >> 4;
    const int64_t block = (int64_t)DT * ps;
    const float* kpool = (const float*)a.c.k;
    const float* vpool = (const float*)a.c.v;
    m = -INFINITY;
    lsum = 0.f;
#pragma unroll
    for (int h = 0; h < DT / 64; ++h) o[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (subs <= 0) return;

    const int head = lane & 3, b = l >> 2, kg = l / (32 / kGroups);
    float q[DT / 16];                                            // step t of the scores takes channels 8 (t / 4) + 4 u + t % 4: block t % 8 of register t / 8
    {
        const float* row = (const float*)a.q + ((int64_t)s * a.hq + (int64_t)g * (a.hq / hkv) + min(head, nh - 1)) * DT;
#pragma unroll
        for (int i = 0; i < DT / 16; ++i) q[i] = row[8 * ((8 * i + b) >> 2) + 4 * u + (b & 3)];
    }
    u32x4 k[DT / 8], v[DT / 8];                                  // k[chunk]; v[(group * 2 + chunk) * kBlocks + channels]
    auto load_k = [&](int i) {
        const int grp0 = (token0 + kStep * i) >> 4, mine = min(kg, last_grp - grp0);         // (a group behind the last one: that again)
        const int pid = __shfl(my_pid, kGroups * i + mine), gi = (grp0 + mine) & gmask;
        const float* kp = kpool + ((int64_t)pid * hkv + g) * block + (gi * 16 + (l & 15)) * 8 + 4 * u;
#pragma unroll
        for (int c = 0; c < DT / 8; ++c) k[c] = load16(kp + (int64_t)c * ps * 8);
    };
    auto load_v = [&](int i) {
        const int grp0 = (token0 + kStep * i) >> 4;
#pragma unroll
        for (int j = 0; j < kGroups; ++j) {
            const int at = min(j, last_grp - grp0);
            const int64_t pid = __builtin_amdgcn_readlane(my_pid, kGroups * i + at);
            const float* vp = vpool + (pid * hkv + g) * block + (int64_t)((grp0 + at) & gmask) * (16 * DT) + l * 8 + 4 * u;
#pragma unroll
            for (int chunk = 0; chunk < 2; ++chunk)
#pragma unroll
                for (int n = 0; n < kBlocks; ++n) v[(j * 2 + chunk) * kBlocks + n] = load16(vp + chunk * (DT * 8) + n * 256);
        }
    };
    load_k(0);
    load_v(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < DT / 16; ++i) q[i] = head < nh ? q[i] : 0.f;
    f32x4 acc_o[kBlocks];                                        // of this half's tokens: channel 32 n + l
#pragma unroll
    for (int n = 0; n < kBlocks; ++n) acc_o[n] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The next sub-step's keys are requested once the score products have taken this one's, its values once the second
    // products have.  (One body with branches: a copy for the last sub-step makes the compiler move the operands about, and spill.)
#pragma unroll 1
    for (int i = 0; i < subs; ++i) {
        const int tok0 = token0 + kStep * i;
        f32x4 acc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        unrolled(std::make_integer_sequence<int, DT / 2>{}, [&](auto c) {
            constexpr int t = c;
            acc[t & 3] = __builtin_amdgcn_mfma_f32_4x4x1f32(q[t / 8], __builtin_bit_cast(f32x4, k[t / 4])[t & 3], acc[t & 3], 3, t % 8, 0);
        });
        if (i + 1 < subs) {
            __builtin_amdgcn_sched_barrier(0);
            load_k(i + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        f32x4 sc;                                                // register = head, lane = token
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float part = (acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]);
            const Two t = swap_halves(part, part);
            sc[e] = t.x + t.y;
        }
        transpose_quads(sc, lane);                               // register = token, lane = head
        const int keep = end - (tok0 + b * 4);
        float xs[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) xs[e] = e < keep ? sc[e] * a.scale : -INFINITY;
        float mx = fmaxf(fmaxf(xs[0], xs[1]), fmaxf(xs[2], xs[3]));
        mx = fmaxf(mx, dpp<kRowRor4>(mx));
        mx = fmaxf(mx, dpp<kRowRor8>(mx));
        const Two two = swap_rows(mx, mx);
        mx = fmaxf(two.x, two.y);
        const float m_new = fmaxf(m, mx);
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = expf(m - m_ref);
        float p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = expf(xs[e] - m_ref);
        lsum = lsum * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
        m = m_new;
#pragma unroll
        for (int e = 0; e < 4; ++e) {                            // where the lower half holds slots 0..7 of a group, the upper holds 8..15
            const int x = __builtin_bit_cast(int, p[e]);
            p[e] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, kRowRor8, 0xC, 0xF, false));
        }
        if (tok0 + kTok > end) {                                 // slots past the last token may hold anything, NaN included
            const int held = end - tok0 - 8 * u;
#pragma unroll
            for (int j = 0; j < 2 * kGroups; ++j)
#pragma unroll
                for (int n = 0; n < kBlocks; ++n)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if ((j >> 1) * 16 + (j & 1) * 4 + e >= held) v[j * kBlocks + n][e] = 0u;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float f = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha), e));
#pragma unroll
            for (int n = 0; n < kBlocks; ++n) acc_o[n][e] *= f;
        }
        unrolled(std::make_integer_sequence<int, 2 * kGroups * 4 * kBlocks>{}, [&](auto c) {
            constexpr int n = c % kBlocks, e = (c / kBlocks) & 3, j = c / (4 * kBlocks);         // channels, token of the quad, (group, chunk)
            constexpr int from = (j >> 1) * 4 + (j & 1);
            acc_o[n] = __builtin_amdgcn_mfma_f32_4x4x1f32(p[e], __builtin_bit_cast(f32x4, v[j * kBlocks + n])[e], acc_o[n], 3, from, 0);
        });
        if (i + 1 < subs) {
            __builtin_amdgcn_sched_barrier(0);
            load_v(i + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int h = 0; h < DT / 64; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const Two t = swap_halves(acc_o[2 * h][e], acc_o[2 * h + 1][e]);
            o[h][e] = t.x + t.y;
        }
    lsum += dpp<kRowRor4>(lsum);
    lsum += dpp<kRowRor8>(lsum);
    const Two two = swap_rows(lsum, lsum);
    lsum = two.x + two.y;
}

// A wave's O of the heads, kChan channels of it, as rows of LDS.
template <int kChan>
__device__ __forceinline__ void few_to_lds(float* rows, const f32x4* o, int lane)
{
#pragma unroll
    for (int h = 0; h < kChan / 64; ++h)
#pragma unroll
        for (int i = 0; i < kFewHeads; ++i) rows[i * kChan + h * 64 + lane] = o[h][i];
}

template <typename E, int DT, bool kExact, bool kFew>
__global__ __launch_bounds__(256, 2) void decode_any_split_kernel(AttnArgs a, int32_t* __restrict__ hdr,
                                                                  float* __restrict__ ws_o, float* __restrict__ ws_ml,
                                                                  int pmax, int head_blocks)
{
    constexpr bool kBf16 = sizeof(E) == 2;
    constexpr int kChan = DT < 128 ? DT : 128;                   // channels the waves' results go through LDS at a time
    __shared__ __attribute__((aligned(16))) float s_o[4][kCols][kChan];
    __shared__ float s_m[4][kCols];
    __shared__ float s_l[4][kCols];
    __shared__ __attribute__((aligned(16))) unsigned char s_q[kCols * q_row<E, DT>()];

    const int B = a.batch, hkv = a.c.hkv, hq = a.hq, G = hq / hkv;
    const int heads = hkv * head_blocks;                         // pairs of a session
    const int D = kExact ? DT : a.c.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x;

    splitk::Share sh;
    if (!splitk::find_share<true>(a.ctx_lens, B, heads, hdr, sh)) return;
    int s = sh.s, base = sh.base, ctx = sh.ctx;
    int n = steps_of(ctx);
    int pair = (sh.f0 - base) / n;                               // (KV head, block of its heads)
    int u = (sh.f0 - base) - pair * n;                           // first step inside the pair

    const int r = lane & 15, c = lane >> 4;
    auto power = [](float x) { return kBf16 ? __builtin_amdgcn_exp2f(x) : expf(x); };

    for (int f = sh.f0; f < sh.f1 && s < B;) {                   // one segment per pass; every value here is uniform
        const int k = min(n - u, sh.f1 - f);
        if (k <= 0) break;                                       // (only if the lengths changed under the kernel)
        const int g = pair / head_blocks, h0 = (pair - g * head_blocks) * kCols;
        const int nh = min(kCols, G - h0);                       // heads of this block
        const int per = (k + 3) >> 2;
        const int my_u = u + w * per;
        const int my_n = max(0, min(per, k - w * per));

        float m, lsum;
        f32x4 o[kFew ? DT / 64 : DT / 16];
        constexpr int kSub = 32 / SubStep<E, DT>::kTok;          // sub-steps of a step
        int my_pid = 0;
        if (my_n > 0) my_pid = a.bt[(int64_t)s * a.max_pages + (min(2 * my_u + lane, (ctx - 1) >> 4) >> (a.c.ps_shift - 4))];
        if constexpr (kFew) {
            constexpr int kTok = kFewTokens;
            attend_few<DT, kTok>(a, s, g, nh, ctx, min(ctx, (my_u + my_n) * 32), my_u * 32, (my_n * 32 + kTok - 1) / kTok, my_pid, m, lsum, o);
        } else {
            queries_to_lds<E, DT, kExact, 256>(a, s, g, h0, nh, s_q);
            attend_steps<E, DT, kExact, 1>(a, g, ctx, my_u * kSub, my_n * kSub, my_pid, s_q, m, lsum, o);
        }

        // o[mb][i] is O^T[channel mb * 16 + c * 4 + i][head r] (kFew: o[h][i] O[head i][channel h * 64 + lane]); the four waves are
        // merged in LDS, kChan channels at a time
        const int first_wg = (base + pair * n) / sh.q;           // the pair's segments are numbered from this workgroup
        const int piece = wg - first_wg;
        if (c == 0) { s_m[w][r] = m; s_l[w][r] = lsum; }        // (kFew: lanes 0..3 hold heads 0..3, the others repeat them)
#pragma unroll
        for (int d0 = 0; d0 < DT; d0 += kChan) {
            if constexpr (kFew) few_to_lds<kChan>(&s_o[w][0][0], o + d0 / 64, lane);
            else
#pragma unroll
                for (int mb = 0; mb < kChan / 16; ++mb) *reinterpret_cast<f32x4*>(&s_o[w][r][mb * 16 + c * 4]) = o[d0 / 16 + mb];
            __syncthreads();
            if (piece < pmax) {
                for (int idx = tid; idx < nh * (kChan / 4); idx += 256) {        // four channels a thread
                    const int head = idx / (kChan / 4), dl = (idx - head * (kChan / 4)) * 4, d = d0 + dl;
                    if (d >= D) continue;
                    float ms = s_m[0][head];                     // wave 0 always has a step: finite unless the scores are not
#pragma unroll
                    for (int ww = 1; ww < 4; ++ww) ms = fmaxf(ms, s_m[ww][head]);
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                    float l = 0.f;
#pragma unroll
                    for (int ww = 0; ww < 4; ++ww) {
                        const float fw = power(s_m[ww][head] - ms);        // a wave without steps has m = -inf -> 0
                        const f32x4 x = *reinterpret_cast<const f32x4*>(&s_o[ww][head][dl]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[e] += fw * x[e];
                        l += fw * s_l[ww][head];
                    }
                    const int64_t slot = ((int64_t)s * hq + (int64_t)g * G + h0 + head) * pmax + piece;
                    *reinterpret_cast<f32x4*>(ws_o + slot * D + d) = acc;
                    if (d == 0) { ws_ml[slot * 2] = ms; ws_ml[slot * 2 + 1] = l; }
                }
            }
            __syncthreads();                                     // s_o, s_m and s_q are written again
        }

        f += k;
        u += k;
        if (u == n) {                                            // on to the next pair
            u = 0;
            if (++pair == heads) {
                pair = 0;
                base += heads * n;
                do {
                    ++s;
                    ctx = s < B ? a.ctx_lens[s] : 0;
                    n = steps_of(ctx);
                } while (s < B && n == 0);
            }
        }
    }
}

// A batch of few, short contexts: one workgroup of eight waves per pair, which shares the pair's steps and writes the
// result itself - no plan, no partials, no merge launch (see one_workgroup_a_pair()).
constexpr int kDirectWaves = 8;
constexpr int kDirectMaxTokens = kDirectWaves * 32 * 32;

// N: channels a thread takes of the waves' results: one while that is one each (half the latency), four beyond.  (Both in one kernel, chosen
// by the pair's heads, cost short calls 0.15 us: 16 sessions of 200 tokens, 32 / 8 heads x 128, 9.57 -> 9.73.)
template <typename E, int DT, bool kExact, int N, bool kFew>
__global__ __launch_bounds__(64 * kDirectWaves, 2) void decode_any_direct_kernel(AttnArgs a, int head_blocks)
{
    constexpr bool kBf16 = sizeof(E) == 2;
    constexpr int kChan = 64, kThreads = 64 * kDirectWaves;
    __shared__ __attribute__((aligned(16))) float s_o[kDirectWaves][kCols][kChan];
    __shared__ float s_m[kDirectWaves][kCols];
    __shared__ float s_l[kDirectWaves][kCols];
    __shared__ uint32_t s_again;                                 // bit h: head h has an element that is not finite
    __shared__ __attribute__((aligned(16))) unsigned char s_q[kCols * q_row<E, DT>()];
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv, D = kExact ? DT : a.c.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int heads = hkv * head_blocks;
    const int s = blockIdx.x / heads, pair = blockIdx.x - s * heads;
    const int g = pair / head_blocks, h0 = (pair - g * head_blocks) * kCols;
    const int nh = min(kCols, G - h0);
    // The wave's sub-steps are every eighth, so that none has more than one over the others (runs of whole steps gave one wave
    // four sub-steps of 16 tokens where three are the most: two fp32 sessions of 300 tokens, 4 / 2 heads x 64, append included, 11.3 ->
    // 9.5 us; 64 of 60 at 32 / 8 x 128 19.8 -> 17.0; bf16 within 1 %), and which they are does not follow from the length: the page ids are fetched beside it.
    constexpr int kTok = kFew ? kFewTokens : SubStep<E, DT>::kTok, kGroups = kTok / 16;
    static_assert(kDirectMaxTokens <= kDirectWaves * (64 / kGroups) * kTok, "the page ids of a wave's sub-steps fit its lanes");
    const int my_pid = a.bt[(int64_t)s * a.max_pages +
                            min((kGroups * (w + kDirectWaves * (lane / kGroups)) + lane % kGroups) >> (a.c.ps_shift - 4), a.max_pages - 1)];
    const int ctx = __builtin_amdgcn_readfirstlane(max(0, min(a.ctx_lens[s], kDirectMaxTokens)));
    const int n = (ctx + kTok - 1) / kTok, subs = w < n ? (n - w - 1) / kDirectWaves + 1 : 0;
    E* out = (E*)a.out + ((int64_t)s * hq + (int64_t)g * G + h0) * D;
    float m, lsum;
    f32x4 o[kFew ? DT / 64 : DT / 16];
    if constexpr (kFew) {
        attend_few<DT, kDirectWaves * kTok>(a, s, g, nh, ctx, ctx, w * kTok, subs, my_pid, m, lsum, o);
    } else {
        queries_to_lds<E, DT, kExact, kThreads>(a, s, g, h0, nh, s_q);
        attend_steps<E, DT, kExact, kDirectWaves>(a, g, ctx, w, subs, my_pid, s_q, m, lsum, o);
    }

    const int r = lane & 15, c = lane >> 4;
    auto power = [](float x) { return kBf16 ? __builtin_amdgcn_exp2f(x) : expf(x); };
    if (c == 0) { s_m[w][r] = m; s_l[w][r] = lsum; }
    if (tid == 0) s_again = 0;
#pragma unroll
    for (int d0 = 0; d0 < DT; d0 += kChan) {
        if (d0 > 0) __syncthreads();
        if constexpr (kFew) few_to_lds<kChan>(&s_o[w][0][0], o + d0 / 64, lane);
        else
#pragma unroll
            for (int mb = 0; mb < kChan / 16; ++mb) *reinterpret_cast<f32x4*>(&s_o[w][r][mb * 16 + c * 4]) = o[d0 / 16 + mb];
        __syncthreads();
        for (int idx = tid; idx < nh * (kChan / N); idx += kThreads) {
            const int head = idx / (kChan / N), dl = (idx - head * (kChan / N)) * N;
            if (d0 + dl >= D) continue;
            float ms = s_m[0][head];                             // wave 0 has a step, if there is one
#pragma unroll
            for (int ww = 1; ww < kDirectWaves; ++ww) ms = fmaxf(ms, s_m[ww][head]);
            float acc[N] = {}, l = 0.f;
#pragma unroll
            for (int ww = 0; ww < kDirectWaves; ++ww) {
                const float fw = power(s_m[ww][head] - ms);      // a wave without steps has m = -inf -> 0
                l += fw * s_l[ww][head];
                typedef float numbers __attribute__((ext_vector_type(N)));
                const numbers x = *reinterpret_cast<const numbers*>(&s_o[ww][head][dl]);
#pragma unroll
                for (int e = 0; e < N; ++e) acc[e] += fw * x[e];
            }
            float trouble = 0.f;
#pragma unroll
            for (int e = 0; e < N; ++e) {
                acc[e] = ctx > 0 ? acc[e] / l : 0.f;
                trouble = general::trouble_of(acc[e], trouble);
            }
            if constexpr (N == 4) splitk::store_quad(out + head * D + d0 + dl, acc);
            else out[head * D + d0 + dl] = (E)acc[0];
            if (!(trouble == 0.f)) atomicOr(&s_again, 1u << head);
        }
    }
    __syncthreads();                                             // (weights in terms turn an infinite sum into NaN)
    const uint32_t all = __builtin_amdgcn_readfirstlane(s_again);
    if (all) general::attend_rows_again<E, 2, (DT + 63) / 64>(a, all & (0x0101u << w), (int64_t)s * hq + (int64_t)g * G + h0 + r, ctx - 1, s, g, &s_o[w][0][0]);
}

// Four channels a lane; a row's lanes lie in one wave, so that a row taken again below is this wave's alone.
__host__ __device__ inline int merge_rows_of_wave(int d) { return 64 / (d >> 2); }

template <typename E>
__global__ __launch_bounds__(256) void decode_any_merge_kernel(AttnArgs a, const int32_t* __restrict__ hdr,
                                                               const float* __restrict__ ws_o,
                                                               const float* __restrict__ ws_ml, int pmax, int head_blocks)
{
    const int D = a.c.d, quads = D >> 2, per_wave = merge_rows_of_wave(D), lane = threadIdx.x & 63;
    const int mine = lane / quads;              // row of the wave; lanes behind the last one have none
    const int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per_wave + mine;        // s * hq + h
    const int s = (int)(row / a.hq), h = (int)(row - (int64_t)s * a.hq), d = (lane - mine * quads) * 4;
    const int ctx = mine < per_wave && row < (int64_t)a.batch * a.hq ? max(a.ctx_lens[s], 0) : -1;      // -1: no row
    E* out = (E*)a.out + row * D;
    float trouble = 0.f;
    if (ctx == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[d + e] = (E)0.0f;
    } else if (ctx > 0) {
        const int G = a.hq / a.c.hkv, g = h / G;
        const int q = max(1, hdr[0]), n = steps_of(ctx);
        const int first = a.c.hkv * head_blocks * hdr[1 + s] + (g * head_blocks + (h - g * G) / kCols) * n;
        const int pieces = min(pmax, (first + n - 1) / q - first / q + 1);   // as the split kernel cuts them
        const f32x4 y = splitk::merge_quad<E, sizeof(E) == 4>(ws_o, ws_ml, row * pmax, pieces, d, D, out);
#pragma unroll
        for (int e = 0; e < 4; ++e) trouble = general::trouble_of(y[e], trouble);
    }
    // (weights in terms, and partials taken with a weight of zero, turn an infinite sum into NaN)
    __shared__ float s_q[4][256];
    uint64_t again = __builtin_amdgcn_ballot_w64(!(trouble == 0.f));
    while (again) {                             // one row at a time
        const int l = __builtin_ctzll(again), r = __builtin_amdgcn_readlane((int)row, l), rs = __builtin_amdgcn_readlane(s, l);
        general::attend_rows_again<E, 1, 4>(a, 1ull << l, row, ctx - 1, rs, (r - rs * a.hq) / (a.hq / a.c.hkv), s_q[threadIdx.x >> 6]);
        again &= ~__builtin_amdgcn_ballot_w64((int)row == r);
    }
}

// Whether every pair, each of at most `bytes` of keys and values, takes one workgroup.  Shares and their merge are two launches
// here (splitk::direct_preferred() weighs the kernel that has a form in one as well), so a workgroup may go through somewhat more: 448
// KiB (432 of fp32 at 64 channels, where a wave has the most sub-steps one behind another), and 1 MiB where the pairs take more than
// half of the CUs, so that shares are hardly finer.  Measured at 256 CUs, append included
// (graph replay), shares -> one workgroup, us, by longest context: one session at 8 / 2 heads, bf16 64 of 1500 tokens 11.8 -> 9.7, of 2200
// 12.3 -> 11.9, of 3500 12.4 -> 15.6; bf16 128 of 600 13.0 -> 10.1, of 1000 13.6 -> 12.2, of 1500 13.6 -> 15.9; fp32 64 of 600 15.2 ->
// 12.0, of 1000 15.8 -> 16.5; 16 at 4 / 4, bf16 128 of 600 14.6 -> 12.4, of 1000 15.3 -> 16.6; fp32 128 of 600 22.5 -> 22.6.  30 at 32 / 8
// (240 pairs): bf16 64 of 2200 24.0 -> 20.6; bf16 128 of 1500 31 -> 28, of 2200 40 -> 37; fp32 128 of 600 33 -> 28, of 1000 43 -> 39,
// of 2200 75 -> 75; bf16 256 of 1000 41 -> 38.  Around the line, shares / one workgroup: fp32 64, 416 to 432 KiB, 0.97 to 1.16, 1.02 over
// 11 batches, 432 to 448 KiB 0.84 to 1.09, 0.92 over 15 (one session of 878 at 4 / 4, 14.0 -> 16.4); bf16 64 and 128, 432 to 448 KiB, 0.85
// to 1.13, 0.98 over 26; rows of 512 bytes and more, 384 to 448 KiB, 1.05 to 1.8.
constexpr int64_t kDirectMostBytes = 1 << 20;
inline bool one_workgroup_a_pair(int64_t pairs, int64_t bytes, bool fp32_64, int cus)
{
    return pairs <= cus && bytes <= (2 * pairs > cus ? kDirectMostBytes : fp32_64 ? 432 << 10 : 448 << 10);
}

// Whether all contexts together come to no more than a share of 256 tokens a CU: shares would leave CUs idle, and walk
// many short contexts one behind the other, where one workgroup per pair (up to eight a CU) takes them side by side.  Measured at
// 256 CUs, shares -> direct, us: 64 sessions at 32 / 8 heads (two pairs a CU) of 32 tokens, bf16 64 21 -> 6.9, bf16 128 27 -> 10.5,
// fp32 128 48 -> 16; of 120 tokens 11.2 -> 7.7, 14.5 -> 12.7, 22.7 -> 20.5; 128 sessions of 60 tokens 15.3 -> 12.8, 19.7 -> 19.7, 33.3 ->
// 33.9, of 120 tokens 13.5 -> 13.4, 18.9 -> 23.7, 32.4 -> 42; 512 sessions of 32 tokens at 4 / 4 heads x 64, 24.8 -> 23.
inline bool few_tokens(int64_t pairs, int max_ctx, int cus)
{
    return pairs <= 8 * cus && max_ctx <= 128 && pairs * max_ctx <= 256 * (int64_t)cus;
}

inline int head_blocks_of(const AttnArgs& a) { return (a.hq / a.c.hkv + kCols - 1) / kCols; }
inline int64_t steps_bound(const AttnArgs& a)
{
    return (int64_t)a.c.hkv * head_blocks_of(a) * a.batch * ((a.max_ctx + 31) / 32);
}

template <typename E, int DT>
ag_status launch(const AttnArgs& a, hipStream_t st)
{
    const int pmax = splitk::pieces_max(a.max_ctx), blocks = head_blocks_of(a);
    const int64_t pair_bytes = (int64_t)a.max_ctx * 2 * DT * (int64_t)sizeof(E);
    static_assert(kDirectMostBytes / (2 * DT * (int)sizeof(E)) <= kDirectMaxTokens, "a wave's page ids fit its lanes");
    const int64_t pairs = (int64_t)a.batch * a.c.hkv * blocks;
    const int cus = stream_cus(st);
    constexpr bool kFewShape = sizeof(E) == 4 && DT <= 128;
    const bool few = kFewShape && a.c.d == DT && a.hq / a.c.hkv <= kFewHeads;
    if (a.max_ctx > 0 && (one_workgroup_a_pair(pairs, pair_bytes, DT == 64 && sizeof(E) == 4, cus) || few_tokens(pairs, a.max_ctx, cus))) {
        const dim3 grid((unsigned)pairs), wg(64 * kDirectWaves);
        prof_before(st);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, wg, 0, st, a, blocks); };
        const bool one = std::min(a.hq / a.c.hkv, kCols) * 64 <= 64 * kDirectWaves;          // channel a thread
        if (few) launch(decode_any_direct_kernel<E, DT, true, 1, kFewShape>);
        else if (a.c.d == DT) one ? launch(decode_any_direct_kernel<E, DT, true, 1, false>) : launch(decode_any_direct_kernel<E, DT, true, 4, false>);
        else one ? launch(decode_any_direct_kernel<E, DT, false, 1, false>) : launch(decode_any_direct_kernel<E, DT, false, 4, false>);
        prof_after(st);
        return hip_check(hipGetLastError(), "decode launch");
    }
    int32_t* hdr = (int32_t*)a.ws;
    float* ws_o = (float*)(hdr + splitk::header_ints(a.batch));
    float* ws_ml = ws_o + (size_t)a.batch * a.hq * pmax * a.c.d;
    prof_before(st);
    if (a.max_ctx > 0) {
        const dim3 grid(share_workgroups(steps_bound(a), st)), wg(256);
        if (few) hipLaunchKernelGGL((decode_any_split_kernel<E, DT, true, kFewShape>), grid, wg, 0, st, a, hdr, ws_o, ws_ml, pmax, blocks);
        else if (a.c.d == DT) hipLaunchKernelGGL((decode_any_split_kernel<E, DT, true, false>), grid, wg, 0, st, a, hdr, ws_o, ws_ml, pmax, blocks);
        else hipLaunchKernelGGL((decode_any_split_kernel<E, DT, false, false>), grid, wg, 0, st, a, hdr, ws_o, ws_ml, pmax, blocks);
        ag_status e = hip_check(hipGetLastError(), "decode split launch");
        if (e) return e;
    }
    const int merge_rows = 4 * merge_rows_of_wave(a.c.d);
    hipLaunchKernelGGL(decode_any_merge_kernel<E>, dim3((unsigned)(((int64_t)a.batch * a.hq + merge_rows - 1) / merge_rows)), dim3(256), 0, st, a, hdr, ws_o, ws_ml, pmax, blocks);
    prof_after(st);
    return hip_check(hipGetLastError(), "decode merge launch");
}

template <typename E>
ag_status launch_for_dim(const AttnArgs& a, hipStream_t st)
{
    if (a.c.d <= 64) return launch<E, 64>(a, st);
    if (a.c.d <= 128) return launch<E, 128>(a, st);
    return launch<E, 256>(a, st);
}

}  // namespace

// Pages below 16 tokens store V transposed without the 8-key chunks these loads rely on, and unaligned pointers rule
// out 16-byte loads: both stay with the general kernel, as do batches whose steps do not fit an int.
bool decode_any_supported(const AttnArgs& a)
{
    return a.c.ps >= 16 && (((uintptr_t)a.q | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 == 0) && steps_bound(a) <= (1 << 30) &&
           (int64_t)a.batch * a.hq <= 0x1fffffff;
}

ag_status launch_decode_any(const AttnArgs& a, hipStream_t st)
{
    return a.c.dtype == AG_BF16 ? launch_for_dim<__bf16>(a, st) : launch_for_dim<float>(a, st);
}

}  // namespace ag
