// Pieces shared by the kernels that deal a batch's contexts in equal shares and merge partials: the decode step and
// the merged decode + short-resume batch (bf16, head_dim 128, page 16: D and PS below), and the decode step of every other
// geometry (attn_decode_any.hip), which takes the plan and the merge.  Internal; not part of the ABI.
#pragma once

#include "ag_internal.h"

namespace ag {
namespace splitk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 128;
constexpr int PS = 16;

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ bf16x8 ld16(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }
// The same load with the streaming hint: K and V are read once per step and never again by this launch, and
// loads marked non-temporal measure 10-15 % more HBM bandwidth on this chip than plain ones.
__device__ __forceinline__ bf16x8 ld16_stream(const __bf16* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p));
}

// v holds 8 tokens: elements 0..3 are tokens j = 0..3, elements 4..7 tokens j = 8..11 of the lane's run.
// Zero element e < 4 unless e < keep_lo, and element 4 + e unless e < keep_hi.
__device__ __forceinline__ bf16x8 keep_quads(bf16x8 v, int keep_lo, int keep_hi)
{
    u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        u[w] &= ((2 * w < keep_lo) ? 0x0000FFFFu : 0u) | ((2 * w + 1 < keep_lo) ? 0xFFFF0000u : 0u);
        u[2 + w] &= ((2 * w < keep_hi) ? 0x0000FFFFu : 0u) | ((2 * w + 1 < keep_hi) ? 0xFFFF0000u : 0u);
    }
    return __builtin_bit_cast(bf16x8, u);
}

struct StepRegs {       // one wave's K and V operands for 32 tokens (two pages)
    bf16x8 k1[4], k2[4], v[8];
};


// Partials that another workgroup of the same launch reads go past this XCD's caches, two floats at a time.
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x2 load_coherent(const float* p)
{
    return __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void store_coherent(float* p, float x, float y)
{
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, f32x2{x, y}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// kNatural: the partials' maxima are in natural units (fp32 caches), not in powers of two.
template <bool kNatural>
__device__ __forceinline__ float merge_power(float x) { return kNatural ? expf(x) : exp2f(x); }

// The partials (m, l, O) of one (row, head), n >= 1 of them: combined in slot order - reproducible - four at a time, with the
// loads of kFlight (4 or 8) in flight together instead of one dependent round trip per partial.  For N neighbouring channels;
// load(i, m, l, o) fetches partial i < n.
template <int N, bool kNatural, int kFlight, class Load>
__device__ __forceinline__ void merge_channels(int n, Load load, float (&out)[N])
{
    float ms = -INFINITY, l = 0.f, acc[N];
#pragma unroll
    for (int e = 0; e < N; ++e) acc[e] = 0.f;
    for (int i0 = 0; i0 < n; i0 += kFlight) {
        float mi[kFlight], li[kFlight], oi[kFlight][N];
#pragma unroll
        for (int h = 0; h < kFlight; h += 4) {
            if (h > 0 && i0 + h >= n) break;
#pragma unroll
            for (int j = h; j < h + 4; ++j) load(min(i0 + j, n - 1), mi[j], li[j], oi[j]);
        }
#pragma unroll
        for (int h = 0; h < kFlight; h += 4) {
            if (h > 0 && i0 + h >= n) break;
#pragma unroll
            for (int j = h; j < h + 4; ++j)
                if (i0 + j >= n) mi[j] = -INFINITY;
            const float m_new = fmaxf(fmaxf(ms, fmaxf(mi[h], mi[h + 1])), fmaxf(mi[h + 2], mi[h + 3]));
            const float keep = ms == -INFINITY ? 0.f : merge_power<kNatural>(ms - m_new);
            l *= keep;
#pragma unroll
            for (int e = 0; e < N; ++e) acc[e] *= keep;
#pragma unroll
            for (int j = h; j < h + 4; ++j) {
                const float f = mi[j] == -INFINITY ? 0.f : merge_power<kNatural>(mi[j] - m_new);     // a partial that saw no key
                l += f * li[j];
#pragma unroll
                for (int e = 0; e < N; ++e) acc[e] += f * oi[j][e];
            }
            ms = m_new;
        }
    }
#pragma unroll
    for (int e = 0; e < N; ++e) out[e] = acc[e] / l;
}

// Four neighbouring channels of a row as E, in one store where the row is aligned for it (uniform: rows are multiples of it apart).
template <typename E>
__device__ __forceinline__ void store_quad(E* out, const float (&y)[4])
{
    typedef E quad __attribute__((ext_vector_type(4)));
    const quad q = {(E)y[0], (E)y[1], (E)y[2], (E)y[3]};
    if ((uintptr_t)out % sizeof(quad) == 0) {
        *reinterpret_cast<quad*>(out) = q;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = q[e];
    }
}

// Channels d .. d + 3 of a (row, head), from partials that other workgroups of the SAME launch wrote (store_coherent): read with device-scope loads, which do not hit in this XCD's caches.  Four channels a thread, 16 bytes of
// a partial in two loads: with one channel a thread a group of 16 heads was eight such chains one after another (step of
// 53 sessions of 750..3260 tokens at 16 / 1 heads 36.4 -> 23.1 us, one session of 8000 at 32 / 8 20.5 -> 15.7, of 1000 8.0 -> 7.4).
__device__ __forceinline__ void merge_coherent(const float* __restrict__ ws_o, const float* __restrict__ ws_ml, int64_t base, int n,
                                               int d, float (&y)[4])
{
    merge_channels<4, false, 8>(n, [&](int i, float& m, float& l, float (&o)[4]) {
        const f32x2 ml = load_coherent(ws_ml + (base + i) * 2);
        const f32x2 lo = load_coherent(ws_o + (base + i) * D + d), hi = load_coherent(ws_o + (base + i) * D + d + 2);
        m = ml[0];
        l = ml[1];
        o[0] = lo[0];
        o[1] = lo[1];
        o[2] = hi[0];
        o[3] = hi[1];
    }, y);
}

// Channels d .. d + 3 of a pair with D_ channels, by the merge kernels: four channels a thread, so that a (row, head) takes
// 32 lanes at 128 channels and 16-byte loads, and a launch a quarter of the workgroups.
template <typename E, bool kNatural = false>
__device__ __forceinline__ f32x4 merge_quad(const float* __restrict__ ws_o, const float* __restrict__ ws_ml, int64_t base, int n,
                                           int d, int D_, E* __restrict__ out)
{
    float y[4];
    merge_channels<4, kNatural, 4>(n, [&](int i, float& m, float& l, float (&o)[4]) {
        m = ws_ml[(base + i) * 2];
        l = ws_ml[(base + i) * 2 + 1];
        const f32x4 x = *reinterpret_cast<const f32x4*>(ws_o + (base + i) * D_ + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = x[e];
    }, y);
    store_quad(out + d, y);
    return f32x4{y[0], y[1], y[2], y[3]};
}

// Workspace is sized for the smallest split a launcher may choose.
constexpr int kMinSplit = 256;

// Workgroup w of W takes steps [w q, (w + 1) q) of the batch's (session, KV head) contexts laid end to end, one step =
// 32 tokens, q = max(kMinSteps, ceil(F / W)).
constexpr int kMinSteps = kMinSplit / 32;      // a workgroup's share is at least this many steps (256 tokens)
constexpr int kMaxSteps = 128;                 // and at most this many (share_workgroups() sizes the grid for it)

__device__ __forceinline__ int steps_of(int ctx) { return ctx > 0 ? (ctx + 31) >> 5 : 0; }

// Segments a pair of n steps starting at flat step a may be cut into when shares are q >= kMinSteps steps.
inline int pieces_max(int max_ctx) { return (((max_ctx + 31) / 32) - 1) / kMinSteps + 2; }
// Workspace: header [q, then the exclusive step count before each session], partials O, partials (m, l).
inline size_t header_ints(int batch) { return ((size_t)batch + 1 + 3) & ~(size_t)3; }

struct Share {
    int q;                  // steps of a share
    int f0, f1;             // this workgroup's steps
    int s, base, ctx;       // session holding step f0, the flat step at which that session starts, its length
};

// Finds this workgroup's share from the lengths (`heads` pairs per session); false if it has none.  Every wave scans the
// lengths for itself, 64 sessions at a time: one memory round trip and no barrier for up to 64 sessions.
// With kPublish workgroup 0 also writes the plan for the merge kernel: hdr[0] = q, hdr[1 + s] = steps before session s.
template <bool kPublish>
__device__ __forceinline__ bool find_share(const int32_t* __restrict__ ctx_lens, int B, int heads, int32_t* __restrict__ hdr,
                                           Share& sh)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wg = blockIdx.x, W = gridDim.x;
    int len = lane < B ? ctx_lens[lane] : 0;
    int total = steps_of(len);
    for (int s = lane + 64; s < B; s += 64) total += steps_of(ctx_lens[s]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) total += __shfl_xor(total, d);
    const int F = heads * __builtin_amdgcn_readfirstlane(total);
    if (F == 0) return false;
    const int q = max(kMinSteps, (F + W - 1) / W);
    const int f0 = wg * q;              // q <= kMaxSteps by the launcher's choice of W: no overflow
    if (kPublish && wg == 0 && tid == 0) hdr[0] = q;
    if (f0 >= F) return false;          // uniform over the workgroup
    sh.q = q;
    sh.f0 = f0;
    sh.f1 = min(f0 + q, F);
    bool found = false;
    int carry = 0;                      // steps of the sessions before this pass of 64
    for (int s0 = 0; s0 < B; s0 += 64) {
        if (s0 > 0) len = s0 + lane < B ? ctx_lens[s0 + lane] : 0;
        const int n = steps_of(len);
        int incl = n;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(f0 < heads * (carry + incl));
        if (!found && hit) {            // the first session that ends behind f0
            const int l = __builtin_ctzll(hit);
            found = true;
            sh.s = s0 + l;
            sh.base = heads * (carry + __builtin_amdgcn_readlane(incl, l) - __builtin_amdgcn_readlane(n, l));
            sh.ctx = __builtin_amdgcn_readlane(len, l);
        }
        if (kPublish && wg == 0 && tid < 64 && s0 + lane < B) hdr[1 + s0 + lane] = carry + incl - n;
        if (found && (!kPublish || wg != 0)) break;      // (uniform; workgroup 0 goes on publishing)
        carry += __builtin_amdgcn_readlane(incl, 63);
    }
    return found;
}

// Whether a decode batch of `pairs` (session, KV head) pairs, each with at most `bytes` of keys and values, takes one
// workgroup per pair and no merge instead of equal shares.  A step of a small batch is a chain of memory round trips, and
// the plan, the partials and their merge are most of them; but beyond 256 KiB a workgroup alone takes 4 to 5 us for every further 256
// KiB, so the longest pair must be short (the host knows no other length), and every pair must have a CU to itself.  416 KiB (832
// tokens of bf16 / 128) is where that turns for few pairs; with more than half of the CUs busy either way, shares are hardly
// finer, and 512 KiB.
// Shares / one workgroup at 256 CUs, graph replay, ag_decode_step and ag_attn_decode with the append.  320 batches of 16 to 256 pairs
// and up to the line, alike, unlike or one session long among short ones: 0.97 to 2.05 up to 832 tokens, 0.88 to 1.53 at 1024 with more
// than 128 pairs (the worst with 200 tokens beside: 17 sessions, 8 KV heads, 11.3 us against 12.9; all of 1024 tokens 19.1 against 15.5).
// Beyond, sessions that are alike still gain, 1.10 to 1.23 up to 1 MiB, but one of 1280, 1536, 2048 tokens among others of 64 or 200 loses:
// 0.76 to 1.06, 0.66 to 0.93, 0.54 to 0.74.  Few pairs at 1024 tokens: 0.67 to 1.55.  Shares come off best where their 256 tokens
// end with the contexts.  (The other shapes have a line of their own, one_workgroup_a_pair() in attn_decode_any.hip.)
inline bool direct_preferred(int64_t pairs, int64_t bytes, int cus)
{
    return pairs <= cus && bytes <= (2 * pairs > cus ? 512 << 10 : 416 << 10);
}

}  // namespace splitk
}  // namespace ag
