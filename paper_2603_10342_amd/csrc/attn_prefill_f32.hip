// Cold and resume prefill over fp32 caches, head_dim 64 or 128, pages of 16 tokens or more, on the bf16 matrix cores.
//
// The fp32 products of the matrix cores run at a sixteenth of the bf16 rate (157 against 2500 TFLOP/s), which is what
// bounds the fp32 form of attn_prefill_any.hip.  Here every fp32 number is taken as three bf16 terms, x = h + m + l
// (each the rounded rest of the ones before: 24 bits and more), and a product as the six of their nine products that
// reach 2^-24 of it: h h + (h m + m h) + (h l + l h + m m).  What is dropped is below 2^-25, less than the rounding of an
// fp32 product; sums are fp32 sums as before.  Terms lie up to 2^-24 below their number and bf16's normal numbers end at
// 2^-126: a number below 2^-102 is off by up to 2^-126 itself.  Columns where that could show are taken again in plain fp32:
// a query with so small a channel, a query so large that a small key counts, an output that small.  Weights, the largest of
// which is about 1, are multiplied by 2^48, so that all down to 2^-126 keep their terms (smaller ones count as zero).
// (Published as bf16x3: Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for
// higher-precision computations", 2019.)  Relative error against 64 bits: 2.4e-7 over four prompts of 300..1500 rows and
// 1.2e-6 over 600 rows on 6000 tokens at 32 / 8 heads x 128; one wave per row, in plain fp32 and in the order of the keys,
// had 3.9e-7 and 1.4e-6.
//
// A workgroup of four waves owns 128 (token, head) columns of one (session, KV head), 32 a wave, whose queries lie in
// registers as terms.  Keys and values are taken 32 at a time: every thread fetches its share of the next tile into
// registers while the current one is multiplied, splits it - once for all four waves - and writes the terms to LDS in
// the layouts of the bf16 kernels, [chunk of 8 channels][key][8] and [chunk of 8 keys][channel][8], two stages.
// Weights are split in registers.  What bounds it is matrix and vector work one after the other: 96 products of 32 clocks a
// tile and wave at 128 channels against 128 of 64, and less than that in softmax, splitting and operand reads.
// Measured, append included, 32 / 8 heads, fp32 products -> terms: four prompts of 300..1500 rows, 128 channels 384 -> 266
// us (135 TFLOP/s of result); eight of 2048, 2510 -> 1630.  Scores in three accumulators and value products grouped by
// term: 3..5 % slower.  The watch on small numbers is 0.4..1.6 % of it, all in the epilogue.
//
// A wave issues in order, and a matrix product behind another holds up the vector work behind it: the weights and the
// splitting are cut into pieces of a few instructions, one behind each product (a pair at once behind every third operand
// before), the maximum of S(t + 1) is taken beside the value product of tile t, and rescaling is outside the tile loop (below).
// 128 channels: 96 products are 46 % of an iteration's clocks, 530 vector instructions 36 %.  Eight prompts of 2048 rows
// 1790 -> 1640 us, eight chunks of 120..300 rows 390 -> 352, 64 channels 852 -> 815 and 212 -> 203; the results are the same
// bits.  Page ids in the lanes of a vector, scalar tile addresses, value products two operands at a time: 2..7 % slower each.
//
// A weight is 2^(s scale log2(e) - m): an exp2, the unit, and two fused products that take a score's two accumulators as
// they are, so that their sum is rounded after m is off it.  Before, e^x as 2^t with the rounding of t put back took seven
// more instructions on an x that had been rounded where it was large.  Four prompts of 300..1500 rows 306 -> 292 us; eight of
// 2048, 128 channels 1912 -> 1827, 64 channels 917 -> 874; eight chunks of 120..300 rows 420 -> 395 and 230 -> 216.  Error
// against 64 bits over 24 batches 0.972 to 0.998 of what it was (with the sum rounded first 0.994 to 1.006).
#include <algorithm>
#include <atomic>

#include "ag_internal.h"
#include "attn_general_row.h"
#include "bf16_terms.h"
#include "tile_list.h"

namespace ag {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kColumns = 128;           // (token, head) pairs of a workgroup
constexpr int BN = 32;                  // keys per tile
constexpr int kRowsAgain = 4;           // rows taken again together (attn_general_row.h)
constexpr float kSlack = 8.0f;          // how far (in powers of two) a maximum may outgrow the reference before O is rescaled

constexpr int plane_bytes(int dt) { return BN * dt * 2; }           // one term of a tile of keys, or of values
constexpr int lds_bytes(int dt) { return 12 * plane_bytes(dt); }    // two stages of K h, m, l, then two of V h, m, l

__device__ __forceinline__ f32x16 product(const u32x4& a, const u32x4& b, const f32x16& c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// unit: scale log2(e), as weights are taken as powers of two
template <int DT>
__global__ __launch_bounds__(256, DT > 64 ? 1 : 2) void prefill_f32_kernel(AttnArgs a, float unit, Deal deal)
{
    constexpr int kPlane = plane_bytes(DT);
    constexpr int kUnits = BN * DT / 8 / 256;       // runs of eight numbers a thread moves of a K tile, and of a V tile
    constexpr int kMb = DT / 32;
    constexpr int kAhead = 4;                       // LDS operand reads run this many operands ahead of their use
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    // ---- which (KV head, session, tile) ----
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv, ps = a.c.ps;
    int g, j;
    if (!place_of(deal, hkv, g, j)) return;
    int s = -1, qt = 0, N = 0, P = 0, row0 = 0;
    find_tile<kColumns>(a, j, G, s, qt, N, P, row0);
    if (s < 0) return;                              // beyond the batch's tiles
    const int ctx = P + N;
    const int col0 = qt * kColumns, cols = min(N * G - col0, kColumns);       // valid columns of the tile
    const Columns columns(col0, G);

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hi = lane >> 5;
    const int cols_w = max(0, min(32, cols - 32 * w));
    const int n_tiles = (P + columns.token(cols - 1)) / BN + 1;               // tiles the workgroup stages
    const int wave_tiles = cols_w > 0 ? (P + columns.token(32 * w + cols_w - 1)) / BN + 1 : 0;     // tiles this wave uses
    const int first_masked = (P + columns.token(32 * w) + 1) / BN;  // first tile holding a key this wave's first column may not see
    const int col = min(32 * w + n, cols - 1);                  // columns beyond the tile repeat the last one
    const int token = columns.token(col);
    const int qpos = P + token;
    const int64_t row = ((int64_t)row0 + token) * hq + (int64_t)g * G + columns.head(col, token);

    // ---- this thread's share of a tile: run i of K is eight channels of a key, of V eight keys of a channel (ag.h) ----
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    const cptr_t bt = (cptr_t)(uintptr_t)(a.bt + (int64_t)s * a.max_pages);
    const int last_grp = (ctx - 1) >> 4, gshift = a.c.ps_shift - 4, gmask = (1 << gshift) - 1;
    const int64_t block = (int64_t)DT * ps;                     // numbers of one (page, head)
    const int key = tid & 31;
    f32x4 kx[kUnits][2], vx[kUnits][2];
    auto fetch_k = [&](int t, int id0, int id1) {               // id0, id1: pages of the tile's two 16-token groups
        const int id = key >> 4 ? id1 : id0, gi = min(2 * t + (key >> 4), last_grp) & gmask;
        const float* kp = (const float*)a.c.k + ((int64_t)id * hkv + g) * block + gi * 128 + (key & 15) * 8;
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const f32x4* p = reinterpret_cast<const f32x4*>(kp + (int64_t)((tid + 256 * i) >> 5) * ps * 8);
            kx[i][0] = p[0];
            kx[i][1] = p[1];
        }
    };
    auto fetch_v = [&](int t, int id0, int id1) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int run = tid + 256 * i, q = run / DT, ch = run % DT;
            const int id = q >> 1 ? id1 : id0, gi = min(2 * t + (q >> 1), last_grp) & gmask;
            const f32x4* p = reinterpret_cast<const f32x4*>((const float*)a.c.v + ((int64_t)id * hkv + g) * block + (int64_t)gi * 16 * DT + ((q & 1) * DT + ch) * 8);
            vx[i][0] = p[0];
            vx[i][1] = p[1];
        }
    };
    auto scrub = [&](int t) {                                   // slots past the last token may hold anything, NaN included
        if (ctx < (t + 1) * BN) {
#pragma unroll
            for (int i = 0; i < kUnits; ++i) {
                const int q = (tid + 256 * i) / DT, keep = ctx - (t * BN + (q >> 1) * 16 + (q & 1) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    vx[i][0][e] = e < keep ? vx[i][0][e] : 0.f;
                    vx[i][1][e] = 8 + e < keep ? vx[i][1][e] : 0.f;
                }
            }
        }
    };
    // What the fetches brought is split a pair at a time, and a pair a term at a time, so that the value product can hide it:
    // pair c of the thread's 8 kUnits (K first), whose run goes to LDS with its last pair.
    Terms run_terms;
    float rest0, rest1;
    auto store_part = [&](int c, int part, unsigned char* k_stage, unsigned char* v_stage) {
        const bool of_v = c >= 4 * kUnits;
        const int i = (c >> 2) % kUnits, e = c & 3;
        const f32x4& src = of_v ? vx[i][e >> 1] : kx[i][e >> 1];
        if (part == 0) {
            rest0 = src[2 * (e & 1)];
            rest1 = src[2 * (e & 1) + 1];
            run_terms.h[e] = take_term(rest0, rest1);
        } else if (part == 1) {
            run_terms.m[e] = take_term(rest0, rest1);
        } else {
            run_terms.l[e] = pack(rest0, rest1);
            if (e == 3) {
                unsigned char* at = (of_v ? v_stage : k_stage) + (tid + 256 * i) * 16;
                *reinterpret_cast<u32x4*>(at) = run_terms.h;
                *reinterpret_cast<u32x4*>(at + kPlane) = run_terms.m;
                *reinterpret_cast<u32x4*>(at + 2 * kPlane) = run_terms.l;
            }
        }
    };
    auto store_pair = [&](int c, unsigned char* k_stage, unsigned char* v_stage) {
#pragma unroll
        for (int part = 0; part < 3; ++part) store_part(c, part, k_stage, v_stage);
    };
    constexpr int kPairs = 8 * kUnits;
    unsigned char* const k_lds = lds;                           // K tile t lives at k_lds + (t & 1) * 3 * kPlane
    unsigned char* const v_lds = lds + 6 * kPlane;              // V tile t lives at v_lds + (t & 1) * 3 * kPlane
    auto id_of = [&](int grp) { return bt[min(grp, last_grp) >> gshift]; };

    // ---- prologue: K(0), V(0) and K(1) into LDS, S(0) ----
    fetch_k(0, id_of(0), id_of(1));
    fetch_v(0, id_of(0), id_of(1));
    // Q^T as B operand: k-step ks covers channels ks * 16 + hi * 8 .. + 7
    Terms qf[DT / 16];
    {
        const float* qp = (const float*)a.q + row * DT + hi * 8;
#pragma unroll
        for (int ks = 0; ks < DT / 16; ++ks) {
            const f32x4* p = reinterpret_cast<const f32x4*>(qp + ks * 16);
            qf[ks] = split8(p[0], p[1]);
        }
    }
    scrub(0);
#pragma unroll
    for (int c = 0; c < kPairs; ++c) store_pair(c, k_lds, v_lds);
    int v0 = id_of(2), v1 = id_of(3), k0 = id_of(4), k1 = id_of(5);           // pages of tiles t + 1 and t + 2 in iteration t
    fetch_k(1, v0, v1);                                       // (past a short context's last group the ids repeat: never used)
#pragma unroll
    for (int c = 0; c < kPairs / 2; ++c) store_pair(c, k_lds + 3 * kPlane, v_lds);

    float m = -INFINITY, lsum = 0.f;
    f32x16 o[kMb];
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mb][i] = 0.f;
    __syncthreads();

    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float x[16], y[16];                                         // S(t) is x + y
    float top[4];                                               // the largest scores of tile t
    auto look = [&](int i) { top[i & 3] = i < 4 ? x[i] + y[i] : fmaxf(top[i & 3], x[i] + y[i]); };
    Terms pf[2];                                                // the weights of tile t
    // S of tile t into s0 + s1 (the h h products, and all smaller ones), with piece(i) of other work behind product i
    constexpr int kProducts = 6 * (DT / 16);                    // of a score tile, and of a value tile
    constexpr int kScoreSteps = 3 * (DT / 16);                  // operand i: k-step i / 3, term i % 3
    auto scores = [&](int t, f32x16& s0, f32x16& s1, auto piece) {
        const unsigned char* kb = k_lds + (t & 1) * 3 * kPlane + hi * 512 + n * 16;
        u32x4 ring[kAhead + 1];
        auto at = [&](int i) { return *reinterpret_cast<const u32x4*>(kb + (i % 3) * kPlane + (i / 3) * 1024); };
#pragma unroll
        for (int i = 0; i < kAhead; ++i) ring[i] = at(i);
#pragma unroll
        for (int i = 0; i < kScoreSteps; ++i) {
            if (i + kAhead < kScoreSteps) ring[(i + kAhead) % (kAhead + 1)] = at(i + kAhead);
            const u32x4 k = ring[i % (kAhead + 1)];
            const Terms& q = qf[i / 3];
            auto add = [&](f32x16& sum, const u32x4& part, int j) {           // product 6 (i / 3) + j
                sum = product(k, part, i == 0 && j < 2 ? zero : sum);
                piece(6 * (i / 3) + j);
                __builtin_amdgcn_sched_barrier(0);
            };
            if (i % 3 == 0) {
                add(s1, q.l, 0);
                add(s0, q.h, 1);
                add(s1, q.m, 2);
            } else if (i % 3 == 1) {
                add(s1, q.m, 3);
                add(s1, q.h, 4);
            } else {
                add(s1, q.h, 5);
            }
        }
    };
    {
        f32x16 s0, s1;
        scores(0, s0, s1, [](int) {});
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            x[i] = s0[i], y[i] = s1[i];
            look(i);
        }
    }
    __syncthreads();                                            // every wave has read K(0): iteration 0 writes K(2) in its place

    // Iteration t: S(t + 1) (matrix) beside the weights P(t) (vector), then O += V(t) . P(t) (matrix) beside the splitting of
    // K(t + 2) and V(t + 1) (vector), which were fetched at its start: one wave per SIMD at 128 channels, so what overlaps is
    // what the wave itself interleaves.  One barrier an iteration: the places it writes, of K(t) and V(t - 1), were last read
    // in iteration t - 1 (K(0) above), before that iteration's barrier.
    // A wave leaves the tile loop where a score outgrew its column's reference maximum, rescales O and enters it again: with
    // the rescaling in the loop the compiler keeps O where vector instructions reach it, and copied the 64 accumulators of 128
    // channels (matrix registers) there and S twice in every iteration, 166 copies, now 64.
#pragma unroll 1
    for (int t = 0;;) {
        float mx = 0.f;
#pragma unroll 1
        for (; t < n_tiles; ++t) {
            const bool mine = t < wave_tiles, next = t + 1 < wave_tiles;
            if (mine) {
                if (t >= first_masked) {                            // the tile straddles this wave's diagonal
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int kk = t * BN + (i >> 2) * 8 + hi * 4 + (i & 3);
                        x[i] = kk <= qpos ? x[i] : -INFINITY;
                        y[i] = kk <= qpos ? y[i] : 0.f;     // (a key not to be seen may be anything, NaN included)
                        look(i);
                    }
                }
                mx = fmaxf(fmaxf(top[0], top[1]), fmaxf(top[2], top[3])) * unit;      // scale > 0: max and scaling commute
                if (__builtin_amdgcn_ballot_w64(mx > m + kSlack) != 0) break;
            }
            const bool more = t + 1 < n_tiles;                      // uniform
            if (more) {
                fetch_v(t + 1, v0, v1);
                fetch_k(t + 2, k0, k1);
                v0 = k0;
                v1 = k1;
                k0 = id_of(2 * (t + 3));
                k1 = id_of(2 * (t + 3) + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (mine) {
                const float m_ref = m == -INFINITY ? 0.f : m;
                float psum[2] = {0.f, 0.f};
                float w0, w1;
                auto weigh = [&](int j, int part) {                 // a sixth of pair j of eight
                    const int i = 2 * j;
                    Terms& to = pf[i >> 3];
                    const int e = (i & 7) >> 1;
                    if (part == 0) {
                        float scale = unit;
                        asm volatile("" : "+s"(scale));             // (here, not all pairs ahead of the products: 4 % of the kernel)
                        w0 = fmaf(y[i], scale, fmaf(x[i], scale, -m_ref));
                        w1 = fmaf(y[i + 1], scale, fmaf(x[i + 1], scale, -m_ref));
                    } else if (part == 1) {
                        w0 = __builtin_amdgcn_exp2f(w0);
                        w1 = __builtin_amdgcn_exp2f(w1);
                    } else if (part == 2) {
                        w0 *= kWeightUnit;
                        w1 *= kWeightUnit;
                        psum[0] += w0;
                        psum[1] += w1;
                    } else if (part == 3) {
                        to.h[e] = take_term(w0, w1);
                    } else if (part == 4) {
                        to.m[e] = take_term(w0, w1);
                    } else {
                        to.l[e] = pack(w0, w1);
                    }
                };
                if (next) {
                    f32x16 s0, s1;
                    scores(t + 1, s0, s1, [&](int i) {              // eight pairs over the score product's steps
                        constexpr int kPer = 6 * 8 / kProducts;     // parts a product: 1 or 2
#pragma unroll
                        for (int k = 0; k < kPer; ++k) weigh((i * kPer + k) / 6, (i * kPer + k) % 6);
                    });
#pragma unroll
                    for (int i = 0; i < 16; ++i) x[i] = s0[i], y[i] = s1[i];
                } else {
#pragma unroll
                    for (int j = 0; j < 48; ++j) weigh(j / 6, j % 6);
                }
                lsum += psum[0] + psum[1];
            }
            unsigned char* const k_to = k_lds + (t & 1) * 3 * kPlane;
            unsigned char* const v_to = v_lds + ((t + 1) & 1) * 3 * kPlane;
            if (more) scrub(t + 1);
            if (mine) {
                const unsigned char* vb = v_lds + (t & 1) * 3 * kPlane + hi * DT * 16 + n * 16;
                constexpr int kN = 6 * kMb;                         // operand i: k-step, term, channel block
                u32x4 ring[kAhead + 1];
                auto at = [&](int i) {
                    return *reinterpret_cast<const u32x4*>(vb + ((i / kMb) % 3) * kPlane + (i / (3 * kMb)) * DT * 32 + (i % kMb) * 512);
                };
#pragma unroll
                for (int i = 0; i < kAhead; ++i) ring[i] = at(i);
#pragma unroll
                for (int i = 0; i < kN; ++i) {
                    if (i + kAhead < kN) ring[(i + kAhead) % (kAhead + 1)] = at(i + kAhead);
                    const u32x4 v = ring[i % (kAhead + 1)];
                    const Terms& p = pf[i / (3 * kMb)];
                    f32x16& acc = o[i % kMb];
                    const int term = (i / kMb) % 3;
                    auto add = [&](const u32x4& part, int j) {       // product 6 kMb (i / 3 kMb) + j
                        const int at = 6 * kMb * (i / (3 * kMb)) + j;
                        acc = product(v, part, acc);
                        if (at < 3 * kPairs) store_part(at / 3, at % 3, k_to, v_to);   // (past the last tile: what is there once more, never read)
                        if (at >= 4 && at < 20) look(at - 4);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    const int b = i % kMb;
                    if (term == 0) {
                        add(p.l, 3 * b);
                        add(p.m, 3 * b + 1);
                        add(p.h, 3 * b + 2);
                    } else if (term == 1) {
                        add(p.m, 3 * kMb + 2 * b);
                        add(p.h, 3 * kMb + 2 * b + 1);
                    } else {
                        add(p.h, 5 * kMb + b);
                    }
                }
                static_assert(3 * kPairs <= kProducts, "the value product's products cover the pairs' parts");
            } else if (more) {
#pragma unroll
                for (int c = 0; c < kPairs; ++c) store_pair(c, k_to, v_to);
            }
            __syncthreads();
        }
        if (t >= n_tiles) break;
        // m is shared by the two lanes of a column: combine them (mx <= m afterwards, or unordered)
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
        lsum *= alpha;
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[mb][i] *= alpha;
        m = m_new;
    }

    // o[mb][q4 * 4 + e] is O^T[channel mb * 32 + q4 * 8 + hi * 4 + e][column n]
    lsum += __shfl_xor(lsum, 32);
    const float inv = 1.0f / lsum;
    // Infinities among Q, K and V come out of the split products as NaN, whatever they would have given (weights times large
    // values may overflow as well); small outputs may have lost terms of theirs.  An output of zero is small too unless its
    // channel is all zeros, so that where there is one the values are looked at once more.
    float trouble = general::trouble_of(inv);
    Least least_o, least_q;
    float most_q = 0.f;
    {
        const float* qp = (const float*)a.q + row * DT + hi * (DT / 2);       // this lane's half of its column's query
#pragma unroll
        for (int i = 0; i < DT / 2; i += 4) {
            const f32x4 q4 = *reinterpret_cast<const f32x4*>(qp + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                least_q.take(q4[e]);
                most_q = fmaxf(most_q, fabsf(q4[e]));
            }
        }
    }
    const bool odd_query = least_q.small() || most_q * a.scale > kLargeQuery;
    uint32_t zero_o = ~0u;
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            trouble = general::trouble_of(o[mb][i], trouble);
            least_o.take(o[mb][i]);
            zero_o = min(zero_o, __builtin_bit_cast(uint32_t, o[mb][i]) << 1);
        }
    const bool zero_out = zero_o == 0 && n < cols_w;
    bool small_values = false;
    uint32_t* const s_any = reinterpret_cast<uint32_t*>(lds + 16 * kRowsAgain * DT);          // [2][wave], behind what attend_rows_again() uses
    auto any_of = [&](bool x, uint32_t* at) {                   // of the workgroup
        const uint64_t lanes = __builtin_amdgcn_ballot_w64(x);
        if (lane == 0) at[w] = lanes != 0;
        __syncthreads();
        return (at[0] | at[1] | at[2] | at[3]) != 0;
    };
    if (any_of(zero_out, s_any)) {
        Least least_v;
        for (int t = 0; t < n_tiles; ++t) {
            fetch_v(t, id_of(2 * t), id_of(2 * t + 1));
            scrub(t);
#pragma unroll
            for (int i = 0; i < kUnits; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) least_v.take(vx[i][e >> 2][e & 3]);
        }
        small_values = any_of(least_v.small(), s_any + 4);
    }
    uint64_t again = __builtin_amdgcn_ballot_w64(n < cols_w && (odd_query || least_o.small(inv) || (zero_out && small_values) || !(trouble == 0.f)));
    again = (again | (again >> 32)) & 0xFFFFFFFFu;              // bit c: column c of this wave
    if (n < cols_w && !((again >> n) & 1)) {
        float* out = (float*)a.out + row * DT + hi * 4;
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = o[mb][q4 * 4 + e] * inv;
                *reinterpret_cast<f32x4*>(out + mb * 32 + q4 * 8) = y;
            }
    }
    general::attend_rows_again<float, kRowsAgain, DT / 64>(a, again, row, qpos, s, g, reinterpret_cast<float*>(lds) + kRowsAgain * DT * w);    // (all are past the last tile)
}

// sum_s ceil(N_s G / 128) <= total G / 128 + batch, and no session has more than ceil(max_new G / 128)
int64_t tiles_bound(const AttnArgs& a)
{
    const int64_t G = a.hq / a.c.hkv;
    return std::min<int64_t>((int64_t)a.total_rows * G / kColumns + a.batch, (int64_t)a.batch * ((a.max_new * G + kColumns - 1) / kColumns));
}

template <int DT>
ag_status launch_kernel(const AttnArgs& a, hipStream_t st)
{
    constexpr int lds = lds_bytes(DT);
    if constexpr (lds > 64 * 1024) {
        static std::atomic<uint64_t> told{0};
        ag_status e = allow_dynamic_lds((const void*)prefill_f32_kernel<DT>, lds, told);
        if (e) return e;
    }
    const float unit = (float)(a.scale * 1.4426950408889634);
    const Deal deal = deal_of(a, tiles_bound(a), stream_cus(st) * (DT > 64 ? 1 : 2) / 8);
    prof_before(st);
    hipLaunchKernelGGL((prefill_f32_kernel<DT>), dim3((unsigned)workgroups_of(deal)), dim3(256), lds, st, a, unit, deal);
    prof_after(st);
    return hip_check(hipGetLastError(), "prefill launch");
}

}  // namespace

bool prefill_f32_supported(const AttnArgs& a)
{
    return a.c.dtype == AG_F32 && (a.c.d == 64 || a.c.d == 128) && a.c.ps >= 16 &&
           (((uintptr_t)a.q | (uintptr_t)a.out | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 == 0) &&
           a.c.hkv * tiles_bound(a) + kDealtPast <= 0x7fffffff && (int64_t)a.total_rows * (a.hq / a.c.hkv) <= 0x7fffffff;
}

ag_status launch_prefill_f32(const AttnArgs& a, hipStream_t st)
{
    return a.c.d == 64 ? launch_kernel<64>(a, st) : launch_kernel<128>(a, st);
}

}  // namespace ag
