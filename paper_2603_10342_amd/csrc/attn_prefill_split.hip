// Prefill of few rows on long contexts (a tool output appended to one agent's session, a handful of short prompts):
// the keys of a query tile are split over the waves of one workgroup.  bf16 and fp32, head_dim 64 and 128, and bf16 at 256;
// pages of 16 tokens or more.
//
// With few rows the other prefill kernels leave the chip idle: a workgroup of 128 columns walks all its keys alone
// (211 rows at 32 / 8 heads are 56 workgroups of 98 key tiles each on 256 CUs).  Here a workgroup owns 32 columns - a
// column is a (token, query head of the group) pair, numbered token * G + head - and its eight waves (four at 256 channels,
// where O^T alone is 128 registers) take every eighth step of 32 keys, each with its own (m, l, O), which are merged through LDS at the end: four times the
// workgroups, each an eighth as long.  Nothing goes through memory between them, so the entry point needs no workspace.
// No wave shares its keys with another, so K and V go straight from the pages into the registers of the matrix
// operands (no LDS stage, no barrier in the loop); K of the next step is requested as soon as the score product has
// read this one's, V after the value product.  What bounds it is the load path of a CU, 64 bytes per clock: a round of
// eight steps at 128 channels, 128 KiB, takes 1.0 us where the same loads alone take 0.9 from L2; scores of the next step
// beside the weights of this one, a second step's keys in flight, or neighbours starting at other steps of a ring of 4 to 16
// all measured slower.  Rest of a call on 6000 tokens (35 us): the append, 8 us of start, merge and launch.  Locating a
// step's pages once for K and V: 36.8 -> 35.1 us there, eight chunks of 50 rows on 2000 tokens 29.0 -> 28.5.  Waits for K and for V
// told apart (the compiler cannot, across the branch around the last requests: a copy of the loop body spills at 128 channels, requests
// without the branch cost a step's traffic): 1.02 to 1.06 at bf16 / 64 on thousands of tokens, 0.97 to 1.0 at bf16 / 128; not taken.
//
// fp32 takes every number as three bf16 terms and a product as six of theirs, as attn_prefill_f32.hip does, with its care for small
// numbers: a step's 128 products of 64 clocks at 128 channels are 96 of 32, beside some 900 vector instructions that split K, V and the
// weights, one wave's behind the other's on a SIMD.  Queries are split once, into LDS.  At 128 channels V is requested when the scores
// are there: a step ahead, 46 registers spill (1.26 times the fp32 products over 30 batches, 1.45 so); four spill as it is, one of them read
// back in every step.  us, fp32 products -> terms, graph
// replay, append included, 32 / 8 heads: 211 rows on 6000 tokens at 128 channels 232 -> 146, 5 rows 221 -> 122, 24 chunks of 20 on 400 75
// -> 54; at 64 channels 125 -> 83, 118 -> 69 and 46 -> 35.  Error against 64 bits over 39 batches 0.46 to 0.80 of what it was.
// The line to the other kernels is at prefill_split_preferred().
#include <algorithm>
#include <atomic>

#include "ag_internal.h"
#include "attn_general_row.h"
#include "bf16_terms.h"
#include "tile_list.h"

namespace ag {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kColumns = 32;            // (token, head) pairs of a workgroup
constexpr int kStep = 32;               // keys of a wave's step
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ f32x16 product(const u32x4& a, const u32x4& b, const f32x16& c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <int DT>
struct Shape {
    static constexpr int waves = DT > 128 ? 4 : 8;          // which share the columns' keys; 512 registers a lane, or 256
    static constexpr int rows_again = DT > 128 ? 1 : 4;     // rows taken again together (attn_general_row.h)
    static constexpr int o_row = DT + 4;                    // floats of a column's partial in LDS, padded
    static constexpr int lds = waves * kColumns * (o_row + 2) * 4 + 16 + 2 * kColumns * 4;
};

// kLo: bf16 weights as three terms (bf16_terms.h); false keeps the rounded weights of the bf16 / 128 / 16 kernels.
// kExact: a wave's reference is the largest score so far, so that the largest weights come out as 1 and lose nothing in rounding, as
// those of the decode queue's own kernels do.  Queues, ten batches: error against 64 bits 0.92 to 0.96 of theirs, where a reference
// that may be outgrown had 0.99 to 1.05; it costs 1 to 10 % of a small queue (rescaling O in most steps).
template <typename E, int DT, bool kLo, bool kExact = false>
__global__ __launch_bounds__((64 * Shape<DT>::waves), (DT > 128 ? 1 : 2)) void prefill_split_kernel(AttnArgs a, Deal deal)
{
    constexpr int kWaves = Shape<DT>::waves, kORow = Shape<DT>::o_row, kRowsAgain = Shape<DT>::rows_again;
    constexpr bool kBf16 = sizeof(E) == 2;
    constexpr int kK = DT * (int)sizeof(E) / 32;    // 16-byte loads of a lane per step: keys
    constexpr int kMb = DT / 32;
    constexpr bool kTakeAgain = kLo || !kBf16;      // columns that are not finite, in plain arithmetic (attn_general_row.h)
    // fp32 at 128 channels: V is requested once the scores are there, not a step ahead; with K, O and the scores' two
    // accumulators it would be more than the registers.
    constexpr bool kLateV = !kBf16 && DT == 128;
    constexpr int kRuns = kBf16 ? 2 : 4;            // runs of keys a lane's weights fall into: 8 keys (bf16), 4 (fp32)
    constexpr bool kQInLds = !kBf16;                // fp32 queries, as three terms, are three times the registers
    constexpr float kSlack = kExact ? 0.f : 8.0f;   // how far a maximum may outgrow the reference before O is rescaled
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];       // Q in the loop (fp32), then the waves' partials

    // ---- which (KV head, session, tile) ----
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv, ps = a.c.ps;
    int g, j;
    if (!place_of(deal, hkv, g, j)) return;
    int s = -1, qt = 0, N = 0, P = 0, row0 = 0;
    find_tile<kColumns>(a, j, G, s, qt, N, P, row0);
    if (s < 0) return;                              // beyond the batch's tiles
    const int ctx = P + N;
    const int col0 = qt * kColumns, cols = min(N * G - col0, kColumns);
    const Columns columns(col0, G);
    auto row_of = [&](int col, int& token) {                    // row (token, head) of Q and O that a column is
        token = columns.token(col);
        return ((int64_t)row0 + token) * hq + (int64_t)g * G + columns.head(col, token);
    };

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int n = lane & 31, hi = lane >> 5;
    const int first_token = columns.token(0), last_token = columns.token(cols - 1);
    int token;
    const int64_t q_row = row_of(min(n, cols - 1), token);      // columns beyond the tile repeat the last one
    const int qpos = P + token;

    const int n_steps = (P + last_token) / kStep + 1;           // of the tile
    const int my_n = w < n_steps ? (n_steps - w - 1) / kWaves + 1 : 0;         // this wave's: steps w, w + 8, ...
    const int first_masked = (P + first_token + 1) / kStep;     // first step holding a key that some column may not see

    // ---- page ids: lane l holds those of own step l / 2 (counted from a multiple of 32), group l % 2 ----
    const int last_grp = (ctx - 1) >> 4, gshift = a.c.ps_shift - 4, gmask = (1 << gshift) - 1;
    const int32_t* const bt = a.bt + (int64_t)s * a.max_pages;
    int my_pid = 0;
    auto fetch_ids = [&](int i) { my_pid = bt[min(2 * (w + kWaves * (i + (lane >> 1))) + (lane & 1), last_grp) >> gshift]; };
    if (my_n > 0) fetch_ids(0);

    // ---- Q^T as B operand: bf16 k-step ks covers channels ks * 16 + hi * 8 .. + 7, fp32 the four channels 4 hi .. of chunks
    // 2 ks and 2 ks + 1, as the loads of K bring them: terms in LDS, [term][ks][hi][column][8] ----
    constexpr int kSteps16 = DT / 16;
    uint32_t* const s_least = reinterpret_cast<uint32_t*>(lds + Shape<DT>::lds) - 2 * kColumns;       // fp32: smallest size in a column's query ...
    uint32_t* const s_most = s_least + kColumns;                                                      // ... and largest
    u32x4 qf[kQInLds ? 1 : kK];
    if constexpr (kQInLds) {
        if (tid < kColumns) {
            s_least[tid] = ~0u;
            s_most[tid] = 0;
        }
        __syncthreads();
        for (int idx = tid; idx < kColumns * kSteps16 * 2; idx += 64 * kWaves) {
            const int c = idx & (kColumns - 1), h = (idx >> 5) & 1, ks = idx >> 6;
            int t;
            const int64_t r = row_of(min(c, cols - 1), t);
            const float* qp = (const float*)a.q + r * DT + ks * 16 + h * 4;
            const f32x4 q0 = *reinterpret_cast<const f32x4*>(qp), q1 = *reinterpret_cast<const f32x4*>(qp + 8);
            const Terms terms = split8(q0, q1);
            *reinterpret_cast<u32x4*>(lds + (((0 * kSteps16 + ks) * 2 + h) * kColumns + c) * 16) = terms.h;
            *reinterpret_cast<u32x4*>(lds + (((1 * kSteps16 + ks) * 2 + h) * kColumns + c) * 16) = terms.m;
            *reinterpret_cast<u32x4*>(lds + (((2 * kSteps16 + ks) * 2 + h) * kColumns + c) * 16) = terms.l;
            Least least;
            float most = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                least.take(q0[e]);
                least.take(q1[e]);
                most = fmaxf(most, fmaxf(fabsf(q0[e]), fabsf(q1[e])));
            }
            atomicMin(s_least + c, least.u);
            atomicMax(s_most + c, __builtin_bit_cast(uint32_t, most));
        }
    } else {
        const E* qp = (const E*)a.q + q_row * DT + hi * 8;
#pragma unroll
        for (int ks = 0; ks < kK; ++ks) qf[ks] = *reinterpret_cast<const u32x4*>(qp + ks * 16);
    }

    const int64_t block = (int64_t)DT * ps;                     // elements of one (page, head)
    u32x4 kx[kK], vx[kRuns * kMb];
    // a step's two groups: elements from a pool's start to their (page, head) blocks, and their places inside them
    struct Groups { int64_t a, b; int ga, gb; };
    auto locate = [&](int i) {                                  // own step i; the steps are located in order
        if ((i & 31) == 0 && i > 0) fetch_ids(i);
        Groups p;
        p.a = ((int64_t)__builtin_amdgcn_readlane(my_pid, 2 * (i & 31)) * hkv + g) * block;
        p.b = ((int64_t)__builtin_amdgcn_readlane(my_pid, 2 * (i & 31) + 1) * hkv + g) * block;
        p.ga = min(2 * (w + kWaves * i), last_grp) & gmask;
        p.gb = min(2 * (w + kWaves * i) + 1, last_grp) & gmask;
        return p;
    };
    auto load_k = [&](const Groups& p) {
        const E* kp = (const E*)a.c.k + (n >> 4 ? p.b + p.gb * 128 : p.a + p.ga * 128) + (n & 15) * 8 + (kBf16 ? hi * ps * 8 : hi * 4);
#pragma unroll
        for (int j = 0; j < kK; ++j) kx[j] = *reinterpret_cast<const u32x4*>(kp + (int64_t)(kBf16 ? 2 * j : j) * ps * 8);
    };
    auto load_v = [&](const Groups& p) {
        const E* vA = (const E*)a.c.v + p.a + p.ga * 16 * DT + (hi * DT + n) * 8;
        const E* vB = (const E*)a.c.v + p.b + p.gb * 16 * DT + (hi * DT + n) * 8;
#pragma unroll
        for (int j = 0; j < kRuns; ++j)
#pragma unroll
            for (int mb = 0; mb < kMb; ++mb)
                vx[j * kMb + mb] = *reinterpret_cast<const u32x4*>((j < kRuns / 2 ? vA : vB) + mb * 32 * 8 + (kBf16 ? 0 : (j & 1) * 4));
    };

    auto hide_v = [&](int st) {                                 // slots past the last token may hold anything, NaN included
        if (ctx < (st + 1) * kStep) {
#pragma unroll
            for (int j = 0; j < kRuns; ++j) {
                const int keep = ctx - (st * kStep + j * (kBf16 ? 16 : 8) + hi * 4);
#pragma unroll
                for (int mb = 0; mb < kMb; ++mb) {
                    u32x4& x = vx[j * kMb + mb];
                    if constexpr (kBf16) {                      // elements 0..3: tokens + j, elements 4..7: + 8 + j
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            x[e] &= (2 * e < keep ? 0xFFFFu : 0u) | (2 * e + 1 < keep ? 0xFFFF0000u : 0u);
                            x[2 + e] &= (2 * e + 8 < keep ? 0xFFFFu : 0u) | (2 * e + 9 < keep ? 0xFFFF0000u : 0u);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = e < keep ? x[e] : 0u;
                    }
                }
            }
        }
    };

    const float unit = a.scale * kLog2e;                        // weights are taken as powers of two
    float m = -INFINITY, lsum = 0.f;
    f32x16 o[kMb];
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mb][i] = 0.f;
    if (kQInLds) __syncthreads();
    Groups at = {};                                             // the step requested last
    if (my_n > 0) {
        at = locate(0);
        load_k(at);
        if (!kLateV) load_v(at);
    }

#pragma unroll 1
    for (int i = 0; i < my_n; ++i) {
        const int st = w + kWaves * i;
        f32x16 sc, rest;                                        // fp32: the score is sc + rest, the products of leading terms and all smaller ones
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = rest[e] = 0.f;
        if constexpr (kBf16) {
#pragma unroll
            for (int j = 0; j < kK; ++j)
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kx[j]), __builtin_bit_cast(bf16x8, qf[j]), sc, 0, 0, 0);
        } else {
#pragma unroll
            for (int ks = 0; ks < kSteps16; ++ks) {
                const unsigned char* at_q = lds + ((ks * 2 + hi) * kColumns + n) * 16;
                constexpr int kTerm = kSteps16 * 2 * kColumns * 16;
                const u32x4 qh = *reinterpret_cast<const u32x4*>(at_q), qm = *reinterpret_cast<const u32x4*>(at_q + kTerm), ql = *reinterpret_cast<const u32x4*>(at_q + 2 * kTerm);
                const Terms k = split8(__builtin_bit_cast(f32x4, kx[2 * ks]), __builtin_bit_cast(f32x4, kx[2 * ks + 1]));
                rest = product(k.h, ql, rest);
                sc = product(k.h, qh, sc);
                rest = product(k.h, qm, rest);
                rest = product(k.m, qm, rest);
                rest = product(k.m, qh, rest);
                rest = product(k.l, qh, rest);
            }
        }
        if (kLateV) {
            __builtin_amdgcn_sched_barrier(0);
            load_v(at);
        }
        if (i + 1 < my_n) {
            at = locate(i + 1);
            load_k(at);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (st >= first_masked) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int key = st * kStep + (e >> 2) * 8 + hi * 4 + (e & 3);
                sc[e] = key <= qpos ? sc[e] : -INFINITY;
                if (!kBf16) rest[e] = key <= qpos ? rest[e] : 0.f;      // (a key not to be seen may be anything, NaN included)
            }
        }
        float mx = kBf16 ? sc[0] : sc[0] + rest[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, kBf16 ? sc[e] : sc[e] + rest[e]);
        mx *= unit;                                             // scale > 0: max and scaling commute
        // m is shared by the two lanes of a column: if either lane's own maximum outgrew it, combine them
        if (__builtin_amdgcn_ballot_w64(mx > m + kSlack) != 0) {
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx);
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
            lsum *= alpha;
#pragma unroll
            for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[mb][e] *= alpha;
            m = m_new;
        }
        const float m_ref = m == -INFINITY ? 0.f : m;           // (a column may see none of this wave's keys so far)
        hide_v(st);
        if constexpr (kBf16) {
            Terms p[2];                                         // (of which only h without kLo)
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[e], unit, -m_ref)), p1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], unit, -m_ref));
                p[e >> 3].set_pair((e & 7) >> 1, p0, p1);
                if constexpr (kLo) {
                    lsum += p0 + p1;
                } else {
                    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
                    lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)p[e >> 3].h[(e & 7) >> 1]), ones, lsum, false);       // the weights as rounded
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mb = 0; mb < kMb; ++mb) {
                    const bf16x8 v = __builtin_bit_cast(bf16x8, vx[j * kMb + mb]);
                    if constexpr (kLo) {
                        o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, __builtin_bit_cast(bf16x8, p[j].l), o[mb], 0, 0, 0);
                        o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, __builtin_bit_cast(bf16x8, p[j].m), o[mb], 0, 0, 0);
                    }
                    o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, __builtin_bit_cast(bf16x8, p[j].h), o[mb], 0, 0, 0);
                }
        } else {
            float psum = 0.f;
            Terms p[2];
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(rest[e], unit, fmaf(sc[e], unit, -m_ref))) * kWeightUnit;
                const float p1 = __builtin_amdgcn_exp2f(fmaf(rest[e + 1], unit, fmaf(sc[e + 1], unit, -m_ref))) * kWeightUnit;
                psum += p0 + p1;
                p[e >> 3].set_pair((e & 7) >> 1, p0, p1);
            }
            lsum += psum;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int mb = 0; mb < kMb; ++mb) {
                    const Terms v = split8(__builtin_bit_cast(f32x4, vx[2 * j * kMb + mb]), __builtin_bit_cast(f32x4, vx[(2 * j + 1) * kMb + mb]));
                    o[mb] = product(v.h, p[j].l, o[mb]);
                    o[mb] = product(v.h, p[j].m, o[mb]);
                    o[mb] = product(v.h, p[j].h, o[mb]);
                    o[mb] = product(v.m, p[j].m, o[mb]);
                    o[mb] = product(v.m, p[j].h, o[mb]);
                    o[mb] = product(v.l, p[j].h, o[mb]);
                }
        }
        if (!kLateV && i + 1 < my_n) load_v(at);
        __builtin_amdgcn_sched_barrier(0);
    }

    // fp32: this wave's keys once more, with fp32 products, where a column's numbers leave the terms' range: a query channel or a result
    // below 2^-100 (zeros aside), values above about 2^70, or what is not finite, which then goes on row by row.  5 rows on 6000 tokens
    // at 32 / 8 heads, one channel of values of 1e-33, row by row -> so: 866 -> 194 us at 64 channels (ordinary values 69, fp32 products
    // alone 118), 1990 -> 367 at 128 (123, 223); an infinite value 980 -> 992 and 2178 -> 2204.  A result of zero only has the values
    // read again, for small ones: 69 -> 81, 123 -> 148.
    auto attend_in_fp32 = [&] {
        asm("" : "+v"(n), "+v"(hi));                         // (nothing is kept in registers for it across the loop above)
        constexpr int kQRow = DT * 4 + 16, kPieces = DT / 4;    // Q in LDS, rows padded
        for (int idx = tid; idx < kColumns * kPieces; idx += 64 * kWaves) {
            const int c = idx / kPieces, p = idx - c * kPieces;
            int t;
            const int64_t r = row_of(min(c, cols - 1), t);
            *reinterpret_cast<u32x4*>(lds + c * kQRow + p * 16) = *reinterpret_cast<const u32x4*>((const float*)a.q + r * DT + p * 4);
        }
        __syncthreads();
        m = -INFINITY;
        lsum = 0.f;
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[mb][e] = 0.f;
        if (my_n > 0) fetch_ids(0);
#pragma unroll 1
        for (int i = 0; i < my_n; ++i) {
            const int st = w + kWaves * i;
            const Groups here = locate(i);
            load_k(here);
            load_v(here);
            f32x16 sc;
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
            for (int j = 0; j < kK; ++j) {
                const f32x4 kf = __builtin_bit_cast(f32x4, kx[j]), q4 = *reinterpret_cast<const f32x4*>(lds + n * kQRow + j * 32 + hi * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], q4[e], sc, 0, 0, 0);
            }
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int key = st * kStep + (e >> 2) * 8 + hi * 4 + (e & 3);
                sc[e] = key <= qpos ? sc[e] : -INFINITY;
                mx = fmaxf(mx, sc[e]);
            }
            mx *= a.scale;
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx), m_ref = m_new == -INFINITY ? 0.f : m_new, alpha = expf(m - m_ref);
            hide_v(st);
            float psum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sc[e] = expf(fmaf(sc[e], a.scale, -m_ref));
                psum += sc[e];
            }
            lsum = lsum * alpha + psum;
            m = m_new;
#pragma unroll
            for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[mb][e] *= alpha;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int mb = 0; mb < kMb; ++mb)
                        o[mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, vx[j * kMb + mb])[e], sc[j * 4 + e], o[mb], 0, 0, 0);
        }
    };

    // ---- the waves' partials through LDS; o[mb][q4 * 4 + e] is O^T[channel mb * 32 + q4 * 8 + hi * 4 + e][column n] ----
    float* const s_o = reinterpret_cast<float*>(lds);           // [wave][column][o_row]
    float* const s_m = s_o + kWaves * kColumns * kORow;
    float* const s_l = s_m + kWaves * kColumns;
    uint32_t* const s_again = reinterpret_cast<uint32_t*>(s_l + kWaves * kColumns);       // bit c: column c is not finite (fp32: or too small); [1]: has a zero; [2]: small values
    auto put_partials = [&] {
        lsum += __shfl_xor(lsum, 32);
        if (kQInLds) __syncthreads();                           // Q has been read
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 x = {o[mb][q4 * 4], o[mb][q4 * 4 + 1], o[mb][q4 * 4 + 2], o[mb][q4 * 4 + 3]};
                *reinterpret_cast<f32x4*>(s_o + (w * kColumns + n) * kORow + mb * 32 + q4 * 8 + hi * 4) = x;
            }
        if (hi == 0) { s_m[w * kColumns + n] = m; s_l[w * kColumns + n] = lsum; }
        if (kTakeAgain && tid < 3) s_again[tid] = 0;
        __syncthreads();
    };
    // Channels d .. d + 7 of columns of `which`: merged, stored, and handed to use() before they are normalised.
    auto merge = [&](uint32_t which, auto power, auto use) {
        for (int idx = tid; idx < cols * (DT / 8); idx += 64 * kWaves) {
            const int c = idx / (DT / 8), d = (idx - c * (DT / 8)) * 8;
            if (!(which >> c & 1)) continue;
            float ms = s_m[c];                                  // wave 0 has the first keys, which every column sees
#pragma unroll
            for (int ww = 1; ww < kWaves; ++ww) ms = fmaxf(ms, s_m[ww * kColumns + c]);
            float l = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ww = 0; ww < kWaves; ++ww) {
                const float f = power(s_m[ww * kColumns + c] - ms);       // a wave that saw no key has m = -inf -> 0
                l += f * s_l[ww * kColumns + c];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += f * s_o[(ww * kColumns + c) * kORow + d + e];
            }
            const float inv = 1.0f / l;
            int t;
            E* out = (E*)a.out + row_of(c, t) * DT + d;
            E y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = (E)(acc[e] * inv);
#pragma unroll
            for (int e = 0; e < (int)sizeof(E) / 2; ++e) reinterpret_cast<u32x4*>(out)[e] = reinterpret_cast<const u32x4*>(y)[e];
            float trouble = general::trouble_of(inv);
#pragma unroll
            for (int e = 0; e < 8; ++e) trouble = general::trouble_of(acc[e], trouble);
            if (kTakeAgain) use(c, d, acc, inv, !(trouble == 0.f));
        }
    };
    put_partials();
    merge(~0u, [](float x) { return __builtin_amdgcn_exp2f(x); }, [&](int c, int d, const float (&acc)[8], float inv, bool again) {
        if constexpr (!kBf16) {                                 // (as in attn_prefill_f32.hip)
            Least least;
            bool zero = false;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                least.take(acc[e]);
                zero |= acc[e] == 0.f;
            }
            again |= least.small(inv);
            if (d == 0) {
                Least least_q;
                least_q.u = s_least[c];
                again |= least_q.small() || __builtin_bit_cast(float, s_most[c]) * a.scale > kLargeQuery;
            }
            if (zero) atomicOr(s_again + 1, 1u << c);
        }
        if (again) atomicOr(s_again, 1u << c);
    });
    if constexpr (kTakeAgain) {
        __syncthreads();                                        // what the waves write once more is behind what is there
        uint32_t all = __builtin_amdgcn_readfirstlane(*s_again);
        if constexpr (!kBf16) {
            const uint32_t zeros = __builtin_amdgcn_readfirstlane(s_again[1]);
            if (zeros) {                                        // uniform over the workgroup: an output of zero is small unless its channel is all zeros
                Least least;
                if (my_n > 0) fetch_ids(0);
                for (int i = 0; i < my_n; ++i) {
                    load_v(locate(i));
                    hide_v(w + kWaves * i);
#pragma unroll
                    for (int j = 0; j < kRuns * kMb; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) least.take(__builtin_bit_cast(f32x4, vx[j])[e]);
                }
                if (least.small()) s_again[2] = 1;
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(s_again[2])) all |= zeros;
            }
            if (all) {
                __syncthreads();                                // (the bits and the partials have been read)
                attend_in_fp32();
                put_partials();
                merge(all, [](float x) { return expf(x); }, [&](int c, int, const float (&)[8], float, bool again) { if (again) atomicOr(s_again, 1u << c); });
                __syncthreads();
                all = __builtin_amdgcn_readfirstlane(*s_again);
            }
        }
        constexpr uint32_t kMine = kWaves == 8 ? 0x01010101u : 0x11111111u;       // columns w, w + kWaves, ...
        int t;
        if (all) general::attend_rows_again<E, kRowsAgain, DT / 64>(a, all & (kMine << w), row_of(min(n, cols - 1), t), qpos, s, g, s_o + kRowsAgain * DT * w);
    }
}

int64_t tiles_bound(const AttnArgs& a, int columns)
{
    const int64_t G = a.hq / a.c.hkv;
    return std::min<int64_t>((int64_t)a.total_rows * G / columns + a.batch, (int64_t)a.batch * ((a.max_new * G + columns - 1) / columns));
}

template <typename E, int DT, bool kLo, bool kExact = false>
ag_status launch_kernel(const AttnArgs& a, hipStream_t st)
{
    constexpr int lds = Shape<DT>::lds;
    static std::atomic<uint64_t> told{0};
    ag_status e = allow_dynamic_lds((const void*)prefill_split_kernel<E, DT, kLo, kExact>, lds, told);
    if (e) return e;
    const Deal deal = deal_of(a, tiles_bound(a, kColumns), stream_cus(st) / 8);
    prof_before(st);
    hipLaunchKernelGGL((prefill_split_kernel<E, DT, kLo, kExact>), dim3((unsigned)workgroups_of(deal)), dim3(64 * Shape<DT>::waves), lds, st, a,
                       deal);
    prof_after(st);
    return hip_check(hipGetLastError(), "prefill launch");
}

}  // namespace

// Whether the batch's query tiles are too few for the other kernels.  Counted in workgroups of 32 columns per CU of the
// stream (one is resident at a time): on long contexts up to 2 for the bf16 / 128 / 16 shape, 3 for the other bf16 shapes, whose
// kernels spend twice the matrix work (weights in three terms), more for fp32, where either kernel is bound by its products.
// Measured at 32 / 8 heads on 256 CUs, append included, the other kernel -> this one: bf16 / 128 / 16, one chunk of
// 5 rows on 6007 tokens (8 workgroups) 114 -> 37 us, 211 rows (216) 119 -> 43, 400 rows (400) 122 -> 77; four chunks of
// 150 rows on 3000 (608) 70 -> 70, eight of 100 on 2000 (832) 57 -> 71.  bf16 / 64 / 64: eight of 40 on 2000 (320) 49 ->
// 32, 32 of 20 on 1000 (768) 32 -> 32, eight of 100 on 2000 (832) 55 -> 58, two prompts of 1000 (2000) 48 -> 54.  bf16 / 256 (graph
// replay): six of 13 rows on 2200 (112) 120 -> 40, eight of 120 on 2000 (784) 119 -> 100, of 160 on 1500 (1024) 100 -> 107.
// A workgroup's start and merge cost it about 8 us whatever its keys, so a second one on a CU pays only where there are keys to
// go through: the line falls to little more than one a CU for the shortest contexts.  Graph replay, this one -> the other: 16 prompts of
// 50 rows (700 workgroups) bf16 / 64 16.1 -> 10.2 us; eight of 100 (660) bf16 / 64
// 15.7 -> 11.6, bf16 / 128 on pages of 32 19.3 -> 15.2, bf16 / 256 29.9 -> 25.4; eight of 50 (360) bf16 / 128 / 16 12.5 -> 11.4;
// four of 200 rows on 300 (630) bf16 / 128 on pages of 32 26.4 -> 23.4; but eight of 60 on 300 (420) bf16 / 64 13.7 ->
// 15.1, 16 of 30 on 600 (490) 16.7 -> 21.2, five of 60 at 16 / 2 (160) bf16 / 128 / 16 8.2 -> 10.5.
// Where a row of bf16 is 512 bytes it rises more slowly: 29 of 101 rows on 274 at 8 / 2 heads (755) bf16 / 256 43 -> 39, 21 of 13 on 25
// (335) 21 -> 17; but eight of 60 on 300 (512) 31 -> 37, 16 of 30 on 600 (512) 39 -> 51.  And there and at fp32 / 128 it does not fall where no
// chunk has more than 32 columns, so that the other kernel has as many workgroups, three quarters empty: 44 of 3 on 32 (352) fp32 / 128
// 23 -> 29.  fp32, over 150 drawn batches, attn_prefill_f32.hip / this one: up to one workgroup a CU 1.0 to 2.8; on a second one
// contexts decide, below 125 tokens at 64 channels 0.72 to 0.97, 125 to 340 1.0 to 1.3, beyond 1.3 to 1.9, at 128 channels below 64 0.69 to
// 0.97, to 250 1.0 to 1.4, beyond 1.4 to 1.7; two to three a CU on 350 to 1750 tokens 1.03 to 1.34, on fewer 0.66 to 0.93; three to five at
// 128 channels on 750 to 1600 1.0 to 1.23, on fewer 0.80 to 1.09; more 0.5 to 0.93.
bool prefill_split_preferred(const AttnArgs& a, bool rounded, hipStream_t st)
{
    if ((a.c.d != 64 && a.c.d != 128 && (a.c.d != 256 || a.c.dtype == AG_F32)) || a.c.ps < 16 || (int64_t)a.total_rows * (a.hq / a.c.hkv) > 0x7fffffff ||
        ((uintptr_t)a.q | (uintptr_t)a.out | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 != 0) return false;
    const int64_t ctx = a.max_ctx;                  // in thousandths of a workgroup per CU:
    const int64_t tiles = tiles_bound(a, kColumns);
    auto between = [](int64_t lo, int64_t x, int64_t hi) { return std::max(lo, std::min(x, hi)); };
    const bool wide = a.c.d * (a.c.dtype == AG_F32 ? 4 : 2) >= 512, one_each = wide && tiles == tiles_bound(a, 128);
    int64_t line;
    if (one_each) line = 3000;
    else if (a.c.dtype == AG_F32 && a.c.d == 64) line = ctx < 125 ? 1000 : between(2000, 2000 + 5 * (ctx - 300), 4000);
    else if (a.c.dtype == AG_F32) line = ctx < 64 ? 1000 : between(2000, 2000 + 5 * (ctx - 200), 5000);
    else if (rounded) line = between(1125, 875 + 2 * ctx, 2000);
    else line = std::min<int64_t>(wide ? 1125 + 4 * ctx : 1250 + 3 * ctx, 3000);
    return 1000 * a.c.hkv * tiles <= line * stream_cus(st);
}

ag_status launch_prefill_split(const AttnArgs& a, bool rounded, hipStream_t st, bool exact)
{
    if (a.c.dtype == AG_F32) return a.c.d == 64 ? launch_kernel<float, 64, false>(a, st) : launch_kernel<float, 128, false>(a, st);
    if (a.c.d == 256) return launch_kernel<__bf16, 256, true>(a, st);
    if (a.c.d == 64) return launch_kernel<__bf16, 64, true>(a, st);
    if (rounded && exact) return launch_kernel<__bf16, 128, false, true>(a, st);
    return rounded ? launch_kernel<__bf16, 128, false>(a, st) : launch_kernel<__bf16, 128, true>(a, st);
}

}  // namespace ag
