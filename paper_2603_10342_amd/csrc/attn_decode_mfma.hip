// Short GQA decode over a paged KV cache, bf16, head_dim 128, page 16
// (paper Sec. II-A: decode reuses the cached keys and values, linear in the
// context; Sec. III-B: one token per active stream per decode step).
//
// The step is bound by HBM: every cached K and V byte is read once
// (2 * Hkv * 128 * 2 B = 4 KiB per token at 8 KV heads) and the arithmetic is
// Hq / Hkv flop per byte.  All G = Hq / Hkv query heads that share a KV head
// are processed together so each byte is fetched once, and the two small
// contractions run on the matrix cores so that the vector ALUs only do the
// softmax bookkeeping.
//
// Work is dealt in equal shares.  The memory system serves the CUs at about equal rates while all of them
// stream, so a launch ends when the CU with the most bytes ends: with one workgroup per (session, head, part of
// the context) the CUs that drew long parts ran up to 45 % over the mean and the step took 112 us where the
// bytes need 95.  Instead, the (session, KV head) pairs are laid end to end in units of one wave step
// (32 tokens, two pages), F steps in all, and workgroup w of W takes steps [w q, (w + 1) q) with
// q = max(8, ceil(F / W)), at most 128: every workgroup, hence every CU, moves the same number of bytes.  A workgroup's
// share covers one pair or the end of one and the start of the next (a "segment" each); every workgroup
// derives the plan itself from the context lengths (a sum and a scan over the batch: the lengths live on
// the device, and a planning launch ahead of this one would cost more than it saves).
//
//   split kernel, per segment: the 4 waves take contiguous quarters and walk them one step at a time, the next step's keys
//   on their way once this one's have been used, and its values likewise:
//     S^T[token][head] = K[token][:] . Q[head][:]     2 x 4 MFMA 16x16x32 (heads padded to 16)
//     streaming softmax on S^T (running max m, running sum l; exp2 with log2(e) folded in)
//     O^T[d][head]    += V^T[d][token] . P^T[token][head]   8 MFMA 16x16x32
//   K rows are loaded straight into the A-operand layout (lane = token row,
//   16 B = 8 channels; pages are chunk-major so 8 neighbouring lanes read 128
//   contiguous bytes); V pages are stored transposed in chunks of 8 keys, so a
//   lane's 16 B load is 8 tokens of one channel, the A operand of the second
//   product.  The MFMA row order of the first product is chosen so that the
//   8 scores a lane ends up with are exactly the 8 tokens its V load covers:
//   no cross-lane shuffles between the products.
//   The 4 waves are merged in LDS and the workgroup writes one partial
//   (m, l, O) per query head and segment to the workspace;
//
//   merge kernel, 32 lanes per (session, query head): combines the partials
//   of the pair's segments in order (reproducible) and writes bf16.
//
// A batch of few, short contexts instead takes one workgroup per pair, which writes its result itself.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "attn_split_common.h"

// Workspace of ag_attn_decode_static: the decode step's header and partials for callers that cannot hand over
// device memory of their own.  One copy per GPU the library runs on, held until the process ends.  In host code
// the name below is only a handle for hipGetSymbolAddress; kernels and copies get the address that call returns.
static __device__ __align__(256) unsigned char scratch[AG_DECODE_STATIC_SCRATCH_BYTES];

namespace ag {

namespace {

using namespace splitk;

// What the whole-step form of the kernel gets on top: the step's new token of every session (one row each),
// which it appends itself, and one counter per (session, KV head), zero on entry and zero again on exit.
struct StepArgs {
    const __bf16* k_new;        // [B][Hkv][D]
    const __bf16* v_new;
    int32_t* counters;          // [B * Hkv]
};

// Every store of this wave up to here has been performed at the scope it was made for.
__device__ __forceinline__ void stores_performed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One wave's part of a segment - steps my_u .. my_u + my_n - 1 of pair (s, g), whose context has ctx tokens: the running
// maximum, the running sum (this lane's share) and O^T of the pair's heads.  appends: this wave's last step is the pair's
// last, and it writes the step's token first.
// kOwnMax: a step's weights stand against the step's own maximum, whose weight is then 1 and loses nothing in rounding, instead of
// against the running one.
template <bool kOwnMax>
__device__ __forceinline__ void attend_steps(const AttnArgs& a, const StepArgs& sa, bool appends, int s, int g, int G, int ctx,
                                             int my_u, int my_n, int lane, float& m, float& lsum, f32x4 (&o)[8])
{
    const int hkv = a.c.hkv, hq = a.hq;
    const __bf16* kpool = (const __bf16*)a.c.k;
    const __bf16* vpool = (const __bf16*)a.c.v;
    const float sl2 = a.scale * kLog2e;
    const int r = lane & 15, c = lane >> 4;
    // Row r of the first score product is slot (r & 7) of page (r >> 3) of the step; the second product takes
    // slots 8..15.  K page layout [chunk][slot][8]: lanes r = 0..7 of one lane group read 128 contiguous bytes.
    // Lane group c then owns slots (c&1)*4 + {0..3} and 8 + (c&1)*4 + {0..3} of page (c >> 1): exactly the 8
    // keys of chunk (c&1) of that value page (see v_offset), so its 16-byte V load is its P operand's partner.
    const int k_pg = r >> 3;
    const int k_off = (c * PS + (r & 7)) * 8;            // + kk * 4 * PS * 8 per k-step; + 8 * 8 for slots 8..15
    const int v_pg = c >> 1;
    const int v_off = ((c & 1) * D + r) * 8;             // value page [half][channel][8 keys]; + mb * 16 * 8 per block

    m = -INFINITY;
    lsum = 0.0f;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) o[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (my_n <= 0) return;

    // Q of the pair's G heads as the B operand: column = head r (zero beyond G), k = channels kk * 32 + c * 8 .. + 7.  Held in
    // registers: a wave waits for no other before its epilogue, and for nothing but page ids before its first keys.
    // Decode step: the segment that ends the pair also appends the step's token (position ctx - 1).  The wave whose
    // part holds the pair's last step writes it - 16 lanes a 16-byte piece of the key each, every lane two
    // channels of the value - once its first step's keys are there, and waits for these stores before it loads that step.
    // Every load of this prologue (page ids, Q, the new token) is issued before the first of them is used.
    bf16x8 qf[4];
    {
        const __bf16* qrow = (const __bf16*)a.q + ((int64_t)s * hq + (int64_t)g * G + min(r, G - 1)) * D + c * 8;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qf[kk] = ld16(qrow + kk * 32);
    }
    const int last_lp = ((ctx + PS - 1) >> 4) - 1;
    // physical pages of a step, clamped to the session's last page; the address is uniform and the table read-only for the
    // kernel's lifetime: scalar loads
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    const cptr_t bt = (cptr_t)(uintptr_t)(a.bt + (int64_t)s * a.max_pages);
    struct Pages { int a, b; };
    auto pages_of = [&](int st) { return Pages{bt[min(2 * (my_u + st), last_lp)], bt[min(2 * (my_u + st) + 1, last_lp)]}; };
    Pages pg = pages_of(0);
    u32x4 new_k = {0, 0, 0, 0};
    __bf16 new_v0 = (__bf16)0.0f, new_v1 = (__bf16)0.0f;
    int64_t last_page = 0;
    if (appends) {
        const __bf16* ks = sa.k_new + ((int64_t)s * hkv + g) * D;
        const __bf16* vs = sa.v_new + ((int64_t)s * hkv + g) * D;
        last_page = bt[last_lp];
        if (lane < 16) new_k = *reinterpret_cast<const u32x4*>(ks + lane * 8);
        new_v0 = vs[lane];
        new_v1 = vs[lane + 64];
    }

    StepRegs x;
    auto load_k = [&](Pages p) {
        const __bf16* kp = kpool + ((int64_t)(k_pg ? p.b : p.a) * hkv + g) * (int64_t)(D * PS) + k_off;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            x.k1[kk] = ld16_stream(kp + kk * 4 * PS * 8);
            x.k2[kk] = ld16_stream(kp + kk * 4 * PS * 8 + 64);
        }
    };
    auto load_v = [&](Pages p) {
        const __bf16* vp = vpool + ((int64_t)(v_pg ? p.b : p.a) * hkv + g) * (int64_t)(D * PS) + v_off;
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) x.v[mb] = ld16_stream(vp + mb * 16 * 8);
    };
    auto append = [&] {
        const int slot = (ctx - 1) & (PS - 1);
        __bf16* kdst = (__bf16*)a.c.k + (last_page * hkv + g) * (int64_t)(D * PS);
        __bf16* vdst = (__bf16*)a.c.v + (last_page * hkv + g) * (int64_t)(D * PS);
        if (lane < 16) *reinterpret_cast<u32x4*>(kdst + (lane * PS + slot) * 8) = new_k;
        vdst[v_offset(slot, lane, PS, D)] = new_v0;
        vdst[v_offset(slot, lane + 64, PS, D)] = new_v1;
    };
    if (appends && my_n == 1) {
        append();
        stores_performed();                              // the token this wave appended lies in the page loaded next
    }
    __builtin_amdgcn_sched_barrier(0);
    load_k(pg);
    load_v(pg);
    pg = pages_of(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        if (r >= G) qf[kk] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};

    // One step; unless it is the wave's last, the next step's keys are requested as soon as the score products have taken
    // this one's, and its values as soon as the second product has: half a step of every wave is always in flight, in the
    // registers of one.  A read of such pages alone takes 173 us for 1183 MB this way and 182 with 16 loads that are waited
    // for together (6.8 and 6.5 TB/s).  64 sessions of 1024..8192 tokens, one launch: 201.5 -> 197 us (1181 MB).
    // Only a wave's last step can reach behind the context.
    auto step = [&](int st, auto last_c) {
        constexpr bool kLast = decltype(last_c)::value;
        const int tok0 = (my_u + st) * 32;
        f32x4 s1 = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.k1[kk], qf[kk], s1, 0, 0, 0);
            s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.k2[kk], qf[kk], s2, 0, 0, 0);
        }
        if constexpr (!kLast) {
            __builtin_amdgcn_sched_barrier(0);
            if (appends && st == 0) append();            // (the first step's keys, requested behind the token, have arrived)
            if (appends && st + 2 == my_n) stores_performed();
            load_k(pg);
            __builtin_amdgcn_sched_barrier(0);
        }
        // s1[i]: token tokb + i, s2[i]: token tokb + 8 + i, of head r
        const int tokb = tok0 + (c >> 1) * PS + (c & 1) * 4;
        const int keep = ctx - tokb;     // token tokb + j exists iff j < keep
        // Rounded before the maximum is taken off (the compiler would make one operation of the two, but not in a wave's last
        // step): equal scores have equal weights wherever they stand, and the maximum's is 1.
        float xs[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma clang fp contract(off)
            xs[i] = !kLast || i < keep ? s1[i] * sl2 : -INFINITY;
            xs[4 + i] = !kLast || 8 + i < keep ? s2[i] * sl2 : -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(xs[0], xs[1]), fmaxf(xs[2], xs[3])), fmaxf(fmaxf(xs[4], xs[5]), fmaxf(xs[6], xs[7])));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);          // finite: token tok0 exists
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        const float m_ref = kOwnMax ? fmaxf(mx, -3e38f) : m_new;          // (scores of -inf: weights of zero)
        const float beta = kOwnMax ? __builtin_amdgcn_exp2f(m_ref - m_new) : 1.f;
        float psum = 0.f;
        bf16x8 pb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(xs[e] - m_ref);
            psum += p;
            pb[e] = (__bf16)p;
        }
        lsum = lsum * alpha + (kOwnMax ? psum * beta : psum);
        m = m_new;
        if (kLast && tok0 + 32 > ctx) {  // last, partial step: unwritten slots may hold anything, NaN included
#pragma unroll
            for (int mb = 0; mb < 8; ++mb) x.v[mb] = keep_quads(x.v[mb], keep, keep - 8);
        }
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
            o[mb] *= alpha;
            if constexpr (kOwnMax)
                o[mb] += beta * __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v[mb], pb, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            else
                o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v[mb], pb, o[mb], 0, 0, 0);
        }
        if constexpr (!kLast) {
            __builtin_amdgcn_sched_barrier(0);
            load_v(pg);
            pg = pages_of(st + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll 1
    for (int st = 0; st + 1 < my_n; ++st) step(st, std::false_type{});
    step(my_n - 1, std::true_type{});
}

// kStep = false: the split half of ag_attn_decode (partials to the workspace, merged by decode_merge_kernel).
// kStep = true: the whole decode step in one launch (ag_decode_step).  The workgroup whose share holds the last
// step of a (session, KV head) pair first writes the step's token into the pair's last page - the wave that will
// read that page does it, and waits for its own stores before it loads the page - and the workgroup that is
// last to finish a pair's segments (an atomic count per pair) merges them, in segment order whoever comes last,
// so the result does not depend on timing; a pair that lies inside one share is normalised and written directly.
template <bool kStep>
__global__ __launch_bounds__(256, 2) void decode_split_kernel(AttnArgs a, int32_t* __restrict__ hdr,
                                                              float* __restrict__ ws_o, float* __restrict__ ws_ml,
                                                              int pmax, StepArgs sa)
{
    __shared__ float s_o[4][16][D];     // per wave, per (padded) head: unnormalised O
    __shared__ float s_m[4][16];
    __shared__ float s_l[4][16];
    __shared__ int s_arrived;           // kStep: how many of the pair's segments had been finished before this one

    const int B = a.batch, hkv = a.c.hkv, hq = a.hq;
    const int G = hq / hkv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x, W = gridDim.x;

    if (kStep) {                        // a session without context gets a row of zeros (no workgroup's share holds it)
        for (int se = wg; se < B; se += W)
            if (a.ctx_lens[se] <= 0)
                for (int idx = tid; idx < hq * D; idx += 256) ((__bf16*)a.out)[(int64_t)se * hq * D + idx] = (__bf16)0.0f;
    }
    Share sh;
    if (!find_share<!kStep>(a.ctx_lens, B, hkv, hdr, sh)) return;
    const int q = sh.q, f0 = sh.f0, f1 = sh.f1;
    int s = sh.s;
    int base = sh.base;                 // flat step at which session s starts
    int ctx = sh.ctx;
    int n = steps_of(ctx);
    int g = (f0 - base) / n;
    int u = (f0 - base) - g * n;        // first step inside (s, g)

    for (int f = f0; f < f1 && s < B;) {                 // one segment per pass; every value here is uniform
        const int k = min(n - u, f1 - f);                // steps of this segment, 1 .. q
        if (k <= 0) break;                               // (only if the lengths changed under the kernel: never spin)
        const int per = (k + 3) >> 2;                    // steps per wave
        const int my_u = u + w * per;
        const int my_n = max(0, min(per, k - w * per));

        const bool appends = kStep && u + k == n && w == (k - 1) / per;        // uniform over the wave
        float m, lsum;
        f32x4 o[8];
        attend_steps<false>(a, sa, appends, s, g, G, ctx, my_u, my_n, lane, m, lsum, o);
        lsum += __shfl_xor(lsum, 16);
        lsum += __shfl_xor(lsum, 32);

        // o[mb][i] is O^T[d = mb*16 + c*4 + i][head r]
        int lane_e = lane, tid_e = tid;                  // (as above: addresses of the merge are computed here)
        asm volatile("" : "+v"(lane_e), "+v"(tid_e));
        const int re = lane_e & 15, ce = lane_e >> 4;
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) *reinterpret_cast<f32x4*>(&s_o[w][re][mb * 16 + ce * 4]) = o[mb];
        if (ce == 0) { s_m[w][re] = m; s_l[w][re] = lsum; }
        __syncthreads();

        // the pair starts at flat step base + g n; its segments are numbered from the workgroup holding that step
        const int first_wg = (base + g * n) / q;
        const int piece = wg - first_wg;
        const int pieces = (base + g * n + n - 1) / q - first_wg + 1;
        const bool direct = kStep && pieces == 1;        // the pair lies inside this share: no partial, no merge
        if (piece < pmax) {
            for (int idx = tid_e; idx < G * (D / 4); idx += 256) {             // four channels a thread
                const int head = idx >> 5, d = (idx & (D / 4 - 1)) * 4;
                float ms = s_m[0][head];               // wave 0 always has a step: finite
#pragma unroll
                for (int ww = 1; ww < 4; ++ww) ms = fmaxf(ms, s_m[ww][head]);
                float l = 0.f;
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ww = 0; ww < 4; ++ww) {
                    const float fw = exp2f(s_m[ww][head] - ms);   // a wave without steps has m = -inf -> 0
                    const f32x4 x = *reinterpret_cast<const f32x4*>(&s_o[ww][head][d]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += fw * x[e];
                    l += fw * s_l[ww][head];
                }
                const int64_t row = (int64_t)s * hq + (int64_t)g * G + head;
                if (direct) {
                    const float y[4] = {acc[0] / l, acc[1] / l, acc[2] / l, acc[3] / l};
                    store_quad((__bf16*)a.out + row * D + d, y);
                } else {
                    const int64_t slot = row * pmax + piece;
                    if (kStep) {                       // read by another workgroup of this launch: device-scope stores
                        store_coherent(ws_o + slot * D + d, acc[0], acc[1]);
                        store_coherent(ws_o + slot * D + d + 2, acc[2], acc[3]);
                        if (d == 0) store_coherent(ws_ml + slot * 2, ms, l);
                    } else {
                        *reinterpret_cast<f32x4*>(ws_o + slot * D + d) = acc;
                        if (d == 0) { ws_ml[slot * 2] = ms; ws_ml[slot * 2 + 1] = l; }
                    }
                }
            }
        }
        if (kStep && !direct) {
            // Count this segment in; whoever completes the pair merges all its segments, in their order.  The
            // partials were stored at device scope (they go past this XCD's caches), every wave waits until its
            // stores have been performed (the barrier by itself orders them only within the workgroup, and does not
            // wait) before the barrier lets the count be raised, and the merging workgroup reads them at device
            // scope after it has seen the full count: no cache-wide write-back or invalidate is needed (a
            // device-wide fence costs a multiple of the whole step here).
            stores_performed();
            __syncthreads();
            if (tid_e == 0) s_arrived = __hip_atomic_fetch_add(&sa.counters[s * hkv + g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (s_arrived == pieces - 1) {
                for (int idx = tid_e; idx < G * (D / 4); idx += 256) {
                    const int head = idx >> 5, d = (idx & (D / 4 - 1)) * 4;
                    const int64_t row = (int64_t)s * hq + (int64_t)g * G + head;
                    float y[4];
                    merge_coherent(ws_o, ws_ml, row * pmax, min(pieces, pmax), d, y);
                    store_quad((__bf16*)a.out + row * D + d, y);
                }
                if (tid_e == 0) sa.counters[s * hkv + g] = 0;      // as the next call expects it
            }
        }
        __syncthreads();                                 // s_o is rewritten by the next segment

        f += k;
        u += k;
        if (u == n) {                                    // on to the next pair
            u = 0;
            if (++g == hkv) {
                g = 0;
                base += hkv * n;
                do {
                    ++s;
                    ctx = s < B ? a.ctx_lens[s] : 0;
                    n = steps_of(ctx);
                } while (s < B && n == 0);
            }
        }
    }
}

// A batch of few, short contexts: one workgroup of 8 waves per (session, KV head) pair, which shares the pair's steps
// and writes the result itself - no plan, no partials, no merge (whose dependent round trips are most of a small step:
// see direct_preferred()).  The waves' results meet in LDS, of which a launch takes what its group size needs.
// (16 waves of 128 registers, all loads of a step waited for together: 32 sessions of 400 tokens, 32 / 8 heads, 11.9 us instead of
// 11.0; 4 of 300 6.25 instead of 5.54.)  With half the waves a part is twice as long; weights against each step's own maximum keep
// the error against 64 bits where that had it (2.00e-3 to 2.06e-3 over 14 batches, 0.98 to 1.0 of it; against the running one 1.01 to 1.023), for
// about 0.1 us (5.43 -> 5.54, 10.98 -> 11.03).
constexpr int kDirectWaves = 8;
constexpr int kDirectMaxTokens = 16 << 10;
inline size_t direct_lds(int G) { return (size_t)kDirectWaves * G * (D + 2) * sizeof(float); }

template <bool kStep>
__global__ __launch_bounds__(64 * kDirectWaves, 2) void decode_direct_kernel(AttnArgs a, StepArgs sa)
{
    extern __shared__ __attribute__((aligned(16))) float s_dyn[];          // [wave][head][D], then m and l [wave][head]
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = blockIdx.x / hkv, g = blockIdx.x - s * hkv;
    const int ctx = min(a.ctx_lens[s], kDirectMaxTokens);
    __bf16* out = (__bf16*)a.out + ((int64_t)s * hq + (int64_t)g * G) * D;
    if (ctx <= 0) {                     // uniform over the workgroup
        for (int idx = tid; idx < G * D; idx += 64 * kDirectWaves) out[idx] = (__bf16)0.0f;
        return;
    }
    const int n = steps_of(ctx), per = (n + kDirectWaves - 1) / kDirectWaves;
    const int my_u = w * per, my_n = max(0, min(per, n - my_u));
    float m, lsum;
    f32x4 o[8];
    attend_steps<true>(a, sa, kStep && w == (n - 1) / per, s, g, G, ctx, my_u, my_n, lane, m, lsum, o);
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
    const int r = lane & 15, c = lane >> 4;
    float* const s_m = s_dyn + kDirectWaves * G * D;
    float* const s_l = s_m + kDirectWaves * G;
    if (r < G) {
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) *reinterpret_cast<f32x4*>(s_dyn + (w * G + r) * D + mb * 16 + c * 4) = o[mb];
        if (c == 0) { s_m[w * G + r] = m; s_l[w * G + r] = lsum; }
    }
    __syncthreads();
    // One channel a thread while that is one each (half the latency), four beyond.
    auto combine = [&](auto channels) {
        constexpr int N = decltype(channels)::value;
        for (int idx = tid; idx < G * (D / N); idx += 64 * kDirectWaves) {
            const int head = idx / (D / N), d = (idx & (D / N - 1)) * N;
            float ms = s_m[head];                               // wave 0 always has a step: finite
#pragma unroll
            for (int ww = 1; ww < kDirectWaves; ++ww) ms = fmaxf(ms, s_m[ww * G + head]);
            float acc[N] = {}, l = 0.f;
#pragma unroll
            for (int ww = 0; ww < kDirectWaves; ++ww) {
                const float fw = exp2f(s_m[ww * G + head] - ms);               // a wave without steps has m = -inf -> 0
                l += fw * s_l[ww * G + head];
                typedef float numbers __attribute__((ext_vector_type(N)));
                const numbers x = *reinterpret_cast<const numbers*>(s_dyn + (ww * G + head) * D + d);
#pragma unroll
                for (int e = 0; e < N; ++e) acc[e] += fw * x[e];
            }
#pragma unroll
            for (int e = 0; e < N; ++e) acc[e] /= l;
            if constexpr (N == 4) store_quad(out + head * D + d, acc);
            else out[idx] = (__bf16)acc[0];
        }
    };
    if (G * D <= 64 * kDirectWaves) combine(std::integral_constant<int, 1>{});
    else combine(std::integral_constant<int, 4>{});
}

constexpr int kMergeRows = 8;               // (session, query head) rows of a merge workgroup, 32 lanes each

__global__ __launch_bounds__(32 * kMergeRows) void decode_merge_kernel(AttnArgs a, const int32_t* __restrict__ hdr,
                                                                       const float* __restrict__ ws_o,
                                                                       const float* __restrict__ ws_ml, int pmax)
{
    const int64_t row = (int64_t)blockIdx.x * kMergeRows + (threadIdx.x >> 5);      // s * hq + h
    if (row >= (int64_t)a.batch * a.hq) return;
    const int s = (int)(row / a.hq), h = (int)(row - (int64_t)s * a.hq);
    const int d = (threadIdx.x & 31) * 4;
    const int ctx = a.ctx_lens[s];
    __bf16* out = (__bf16*)a.out + row * D;
    if (ctx <= 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[d + e] = (__bf16)0.0f;
        return;
    }
    const int q = max(1, hdr[0]), n = steps_of(ctx);
    const int first = a.c.hkv * hdr[1 + s] + (h / (a.hq / a.c.hkv)) * n;       // the pair's first flat step
    const int pieces = min(pmax, (first + n - 1) / q - first / q + 1);          // as the split kernel cuts them
    merge_quad(ws_o, ws_ml, row * pmax, pieces, d, D, out);
}

}  // namespace

// CUs of the current device.
int device_cus()
{
    static std::atomic<int> cached[16];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return 256; }
    const bool in_table = dev >= 0 && dev < 16;
    if (in_table) { const int v = cached[dev].load(); if (v > 0) return v; }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        cus = 256;
    }
    if (in_table) cached[dev].store(cus);
    return cus;
}

// CUs the stream's launches may use: the bits of its CU mask (paper Sec. III-C: decode runs on a partition),
// the whole device if the stream has none.
int stream_cus(hipStream_t st)
{
    const int all = device_cus();
    uint32_t words[32] = {0};
    const uint32_t n_words = (uint32_t)std::min(32, (all + 31) / 32);
    if (hipExtStreamGetCUMask(st, n_words, words) != hipSuccess) { (void)hipGetLastError(); return all; }
    int n = 0;
    for (uint32_t i = 0; i < n_words; ++i) n += __builtin_popcount(words[i]);
    return n > 0 && n <= all ? n : all;
}

// Workgroups of a launch: the shares are equal, so what matters is that every CU gets the same number of them, and as few as the
// longest share (kMaxSteps) allows: each workgroup pays the plan and each segment a read of page ids (two per CU measured 1.5 %
// faster than four, and a grid that leaves some CUs one workgroup short loses 4-5 %).  At most kMaxSteps: in attn_decode_any.hip a lane
// holds a page id; here the largest weight of a wave's part is 1 and loses nothing in rounding, and longer parts have fewer of
// them.  64 sessions of 1024..8192 tokens in two workgroups a CU whatever their shares, in this many: 194 / 197 us (1 to 4 % over 15
// batches of long contexts), error against 64 bits 2.185e-3 / 2.168e-3.
int share_workgroups(int64_t f_max, hipStream_t st)
{
    const int64_t unit = 2 * (int64_t)stream_cus(st);
    const int64_t need = std::max<int64_t>(1, (f_max + kMaxSteps - 1) / kMaxSteps);
    return (int)(unit * ((need + unit - 1) / unit));
}

size_t decode_workspace_bytes(int batch, int hq, int d, int max_ctx)
{
    if (batch <= 0) return 0;
    return header_ints(batch) * sizeof(int32_t) + (size_t)batch * hq * pieces_max(max_ctx) * (size_t)(d + 2) * sizeof(float);
}

bool decode_mfma_supported(const AttnArgs& a)
{
    return a.c.dtype == AG_BF16 && a.c.d == D && a.c.ps == PS && (a.hq / a.c.hkv) <= 16 &&
           (((uintptr_t)a.q | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 == 0);
}

ag_status decode_static_scratch(void** ptr_out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    int dev = -1;
    ag_status e = hip_check(hipGetDevice(&dev), "hipGetDevice");
    if (e) return e;
    if (dev < 0 || dev >= kMaxDevices) { set_error("device %d is beyond the %d devices the static scratch is kept for", dev, kMaxDevices); return AG_ERR_UNSUPPORTED; }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {                   // each device holds its own copy of the array at its own address
        void* p = nullptr;
        if ((e = hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)"))) return e;
        if (!p) { set_error("hipGetSymbolAddress(scratch) returned a null address"); return AG_ERR_HIP; }
        ptrs[dev] = p;
    }
    *ptr_out = ptrs[dev];
    return AG_OK;
}

// The same rule for ag_attn_decode and ag_decode_step: their results are bit for bit the same.
static bool takes_direct(const AttnArgs& a, hipStream_t st)
{
    return a.max_ctx > 0 && direct_preferred((int64_t)a.batch * a.c.hkv, (int64_t)a.max_ctx * 4 * D, stream_cus(st));
}

template <bool kStep>
static ag_status launch_direct(const AttnArgs& a, const StepArgs& sa, hipStream_t st)
{
    static std::atomic<uint64_t> told{0};
    const size_t lds = direct_lds(a.hq / a.c.hkv);
    if (lds > 64 * 1024) {                          // (groups of 8 heads and more)
        ag_status e = allow_dynamic_lds((const void*)decode_direct_kernel<kStep>, (int)direct_lds(16), told);
        if (e) return e;
    }
    prof_before(st);
    hipLaunchKernelGGL(decode_direct_kernel<kStep>, dim3(a.batch * a.c.hkv), dim3(64 * kDirectWaves), lds, st, a, sa);
    prof_after(st);
    return hip_check(hipGetLastError(), "decode launch");
}

ag_status launch_decode_mfma(const AttnArgs& a, void* ws, hipStream_t st)
{
    if (takes_direct(a, st)) return launch_direct<false>(a, StepArgs{}, st);
    const int pmax = pieces_max(a.max_ctx);
    int32_t* hdr = (int32_t*)ws;
    float* ws_o = (float*)(hdr + header_ints(a.batch));
    float* ws_ml = ws_o + (size_t)a.batch * a.hq * pmax * D;
    // Upper bound of the step count from the host-known bounds; the grid is sized so that a share is at most
    // kMaxSteps steps even if every session is max_ctx long.
    const int64_t f_max = (int64_t)a.c.hkv * a.batch * ((a.max_ctx + 31) / 32);
    if (f_max > (1 << 30)) { set_error("decode batch of %lld steps of 32 tokens is beyond one launch", (long long)f_max); return AG_ERR_INVALID_ARG; }
    if (a.max_ctx > 0) {
        const int grid = share_workgroups(f_max, st);
        // the event bracket covers both kernels of the call: the merge kernel writes the output the byte count includes
        prof_before(st);
        hipLaunchKernelGGL(decode_split_kernel<false>, dim3(grid), dim3(256), 0, st, a, hdr, ws_o, ws_ml, pmax, StepArgs{});
        ag_status e = hip_check(hipGetLastError(), "decode split launch");
        if (e) return e;
    }
    hipLaunchKernelGGL(decode_merge_kernel, dim3((unsigned)(((int64_t)a.batch * a.hq + kMergeRows - 1) / kMergeRows)), dim3(32 * kMergeRows), 0, st, a, hdr, ws_o, ws_ml, pmax);
    prof_after(st);
    return hip_check(hipGetLastError(), "decode merge launch");
}

// ---- the whole step in one launch ----
// Workspace: a counter region of fixed size at the start - wherever the partials of a call of another shape
// may have landed, they never land here, so the counters stay zero from call to call - then the split
// kernel's workspace.
static size_t step_counter_bytes(int, int) { return AG_DECODE_STEP_COUNTER_BYTES; }

size_t decode_step_workspace_bytes(int batch, int hq, int d, int max_ctx)
{
    if (batch <= 0) return 0;
    return step_counter_bytes(batch, hq) + decode_workspace_bytes(batch, hq, d, max_ctx);
}

ag_status launch_decode_step(const AttnArgs& a, const void* k_new, const void* v_new, void* ws, hipStream_t st)
{
    if ((int64_t)a.batch * a.c.hkv * (int64_t)sizeof(int32_t) > (int64_t)AG_DECODE_STEP_COUNTER_BYTES) {
        set_error("batch * num_kv_heads = %lld exceeds the %d counters of a decode-step workspace", (long long)a.batch * a.c.hkv,
                  (int)(AG_DECODE_STEP_COUNTER_BYTES / sizeof(int32_t)));
        return AG_ERR_INVALID_ARG;
    }
    const int pmax = pieces_max(a.max_ctx);
    int32_t* counters = (int32_t*)ws;
    int32_t* hdr = (int32_t*)((unsigned char*)ws + step_counter_bytes(a.batch, a.hq));
    float* ws_o = (float*)(hdr + header_ints(a.batch));
    float* ws_ml = ws_o + (size_t)a.batch * a.hq * pmax * D;
    const int64_t f_max = (int64_t)a.c.hkv * a.batch * ((a.max_ctx + 31) / 32);
    if (f_max > (1 << 30)) { set_error("decode batch of %lld steps of 32 tokens is beyond one launch", (long long)f_max); return AG_ERR_INVALID_ARG; }
    if (takes_direct(a, st)) return launch_direct<true>(a, StepArgs{(const __bf16*)k_new, (const __bf16*)v_new, counters}, st);
    const int grid = share_workgroups(std::max<int64_t>(f_max, 1), st);
    prof_before(st);
    hipLaunchKernelGGL(decode_split_kernel<true>, dim3(grid), dim3(256), 0, st, a, hdr, ws_o, ws_ml, pmax,
                       StepArgs{(const __bf16*)k_new, (const __bf16*)v_new, counters});
    prof_after(st);
    return hip_check(hipGetLastError(), "decode step launch");
}

}  // namespace ag
