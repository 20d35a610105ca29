// Cold and resume prefill over paged KV caches of any supported head_dim and dtype with pages of 16 tokens or more
// (bf16 at head_dim 128, and at 64 on long contexts, takes attn_prefill_mfma.hip, see prefill_mfma_lo_supported(); fp32 at
// 64 and 128 takes attn_prefill_f32.hip; few rows take attn_prefill_split.hip).
//
// A dense contraction, bound by the matrix cores.  A workgroup of four waves owns 128 columns of one (session, KV
// head): a column is a (token, query head of the group) pair, numbered token * G + head, so that any group size fills
// its tiles; a wave owns 32 columns and keeps their Q in registers.  Keys and values are taken BN at a time (64 for
// bf16, 32 for fp32: 128 * DT bytes each) through two LDS stages by direct global-to-LDS loads, requested one tile
// ahead; two workgroups per CU (head_dim up to 128) cover each other's softmax and barriers.
//   S^T[key][column] = K . Q^T, online softmax under a reference maximum, O^T[channel][column] += V^T . P^T
// on 32x32x16 (bf16) and 32x32x2 (fp32) products.  The score layout's rows are the keys a lane owns, four in a run,
// and both pools store those runs contiguously (ag.h), so P stays in registers in both types.
// Precision: fp32 runs in fp32 throughout (expf, fp32 products: 157 TFLOP/s at most); bf16 caches multiply the weights
// as three bf16 terms (bf16_terms.h), twice the matrix work, so that they stay in 32 bits: two terms, 16 bits, take 268 us
// instead of 336 for the prompts below, and are off from 64 bits by 1e-6 more of the error that the rounding of outputs makes.
// Measured, append included (one wave per (row, query head) before -> now): eight bf16 prompts of 2048 rows at 32 / 8 heads
// x 64, 64-token pages, 57 -> 0.336 ms (410 TFLOP/s of result, 820 of products).
#include <algorithm>
#include <atomic>

#include "ag_internal.h"
#include "attn_general_row.h"
#include "bf16_terms.h"
#include "lds_dma.h"
#include "tile_list.h"

namespace ag {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kColumns = 128;           // (token, head) pairs of a workgroup
constexpr float kLog2e = 1.4426950408889634f;
// rows taken again together (attn_general_row.h); 256 channels have no registers to spare (2 % of the kernel)
constexpr int rows_again(int dt) { return dt > 128 ? 1 : 4; }
constexpr int kAhead = 3;               // LDS operand reads run this many operands ahead of their use

// use(i, operand i) for i = 0 .. N - 1, operand i read from at(i) kAhead operands before its use
template <int N, class At, class Use>
__device__ __forceinline__ void with_operands(At at, Use use)
{
    u32x4 ring[kAhead + 1];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) ring[i] = *reinterpret_cast<const u32x4*>(at(i));
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (i + kAhead < N) ring[(i + kAhead) % (kAhead + 1)] = *reinterpret_cast<const u32x4*>(at(i + kAhead));
        use(i, ring[i % (kAhead + 1)]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <typename E, int DT, bool kExact>
__global__ __launch_bounds__(256, DT > 128 ? 1 : 2) void prefill_any_kernel(AttnArgs a, Deal deal)
{
    constexpr bool kBf16 = sizeof(E) == 2;
    constexpr int BN = 128 / (int)sizeof(E);        // keys per tile
    constexpr int kTile = 128 * DT;                 // bytes of a K tile, and of a V tile
    constexpr int kPer = DT / 32;                   // direct loads of a wave for a K tile, and for a V tile
    constexpr int kGroups = BN / 16;                // 16-token groups of a tile
    constexpr int kScores = BN / 2;                 // scores a lane holds (its partner lane ^ 32 holds the other half)
    // a reference maximum may be outgrown by this much before O is rescaled (8 in powers of two, as fp32 has range)
    constexpr float kSlack = kBf16 ? 8.0f : 5.5f;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];       // [2 stages][K tile, V tile]

    // ---- which (KV head, session, tile) ----
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv;
    const int D = kExact ? DT : a.c.d, ps = a.c.ps;
    int g, j;
    if (!place_of(deal, hkv, g, j)) return;
    int s = -1, qt = 0, N = 0, P = 0, row0 = 0;
    find_tile<kColumns>(a, j, G, s, qt, N, P, row0);
    if (s < 0) return;                              // beyond the batch's tiles
    const int ctx = P + N;
    const int col0 = qt * kColumns, cols = min(N * G - col0, kColumns);       // valid columns of the tile
    const Columns columns(col0, G);

    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int wu = __builtin_amdgcn_readfirstlane(w);           // the same value, known to be uniform
    const int n = lane & 31, hi = lane >> 5;
    const int cols_w = max(0, min(32, cols - 32 * wu));
    const int last_token = columns.token(cols - 1);
    const int n_tiles = (P + last_token) / BN + 1;                            // tiles the workgroup stages
    const int wave_tiles = cols_w > 0 ? (P + columns.token(32 * wu + cols_w - 1)) / BN + 1 : 0;     // tiles this wave uses
    const int first_masked = (P + columns.token(32 * wu) + 1) / BN;  // first tile holding a key this wave's first column may not see

    const int col = min(32 * w + n, cols - 1);                  // columns beyond the tile repeat the last one
    const int token = columns.token(col), head = columns.head(col, token);
    const int qpos = P + token;
    const int64_t row = ((int64_t)row0 + token) * hq + (int64_t)g * G + head;

    // ---- Q^T as B operand: bf16 k-step ks covers channels ks * 16 + hi * 8 .. + 7, fp32 chunk j channels 8 j + hi * 4 .. + 3
    constexpr int kQ = kBf16 ? DT / 16 : DT / 8;
    u32x4 qf[kQ];
    {
        const unsigned char* qp = (const unsigned char*)a.q + row * D * (int)sizeof(E) + hi * 16;
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const bool in = kExact || i * 32 + hi * 16 < D * (int)sizeof(E);
            qf[i] = u32x4{0, 0, 0, 0};
            if (in) qf[i] = *reinterpret_cast<const u32x4*>(qp + i * 32);
        }
    }

    // ---- tile requests ----
    // Page ids by scalar loads (the index is uniform), fetched an iteration before the tile's data is requested.
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    const cptr_t bt = (cptr_t)(uintptr_t)(a.bt + (int64_t)s * a.max_pages);
    const int last_grp = (ctx - 1) >> 4, gshift = a.c.ps_shift - 4, gmask = (1 << gshift) - 1;
    const int64_t block = (int64_t)D * ps;                      // elements of one (page, head)
    const int k_grp = kBf16 ? lane >> 4 : (lane & 31) >> 4;     // this lane's group of a K tile
    const int v_grp = kBf16 ? wu : wu >> 1;                     // this wave's group of a V tile
    struct Pages { int k, v; };
    auto pages_of = [&](int t, Pages& pg) {
        pg.k = 0;
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {                     // this lane's page among the tile's (uniform) ids, by masks
            const int id = bt[min(t * kGroups + i, last_grp) >> gshift];
            pg.k |= id & (k_grp == i ? -1 : 0);
        }
        pg.v = bt[min(t * kGroups + v_grp, last_grp) >> gshift];
    };
    // K tile: bf16 [chunk of 8 channels][64 keys][8], fp32 [half chunk][32 keys][4]: one load moves a chunk of all keys.
    // V tile: 16-byte pieces [bf16: chunk of 8 keys, fp32: quad of 4 keys][channel]; the wave's loads lie in one group.
    auto request = [&](int t, int stage, const Pages& pg) {
        const int gk = min(t * kGroups + k_grp, last_grp) & gmask, gv = min(t * kGroups + v_grp, last_grp) & gmask;
        const unsigned k_dst = lds_address(lds) + stage * 2 * kTile + (wu * kPer) * 1024;
        const E* kp = (const E*)a.c.k + ((int64_t)pg.k * hkv + g) * block + (gk * 16 + (lane & 15)) * 8 + (kBf16 ? 0 : hi * 4);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int chunk = wu * kPer + i;
            if (kExact || chunk * 8 < D) load_to_lds(kp + (int64_t)chunk * ps * 8, k_dst + i * 1024);    // (zeroed below otherwise)
        }
        const unsigned v_dst = lds_address(lds) + stage * 2 * kTile + kTile + (wu * kPer) * 1024;
        const E* vp = (const E*)a.c.v + ((int64_t)__builtin_amdgcn_readfirstlane(pg.v) * hkv + g) * block + gv * 16 * D;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int unit = (wu * kPer + i) / (DT / 64), ch0 = ((wu * kPer + i) % (DT / 64)) * 64;     // chunk or quad of the tile
            const int ch = kExact ? ch0 + lane : min(ch0 + lane, D - 1);
            const int at = kBf16 ? ((unit & 1) * D + ch) * 8 : ((unit & 1) * D + ch) * 8 + ((unit >> 1) & 1) * 4;
            load_to_lds(vp + at, v_dst + i * 1024);
        }
    };
    // Slots behind the session's last token may hold anything (NaN included) and would poison the value product even
    // under a zero weight: once the wave's part of V(t) has landed, zero them.
    auto scrub_v = [&](int t, int stage) {
        if (ctx < (t + 1) * BN) {                               // uniform
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int unit = (wu * kPer + i) / (DT / 64);
                u32x4* p = reinterpret_cast<u32x4*>(lds + stage * 2 * kTile + kTile + (wu * kPer + i) * 1024 + lane * 16);
                u32x4 x = *p;
                if constexpr (kBf16) {                          // elements 0..3: tokens tok + j, elements 4..7: tok + 8 + j
                    const int keep = ctx - (t * BN + (unit >> 1) * 16 + (unit & 1) * 4);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        x[j] &= (2 * j < keep ? 0xFFFFu : 0u) | (2 * j + 1 < keep ? 0xFFFF0000u : 0u);
                        x[2 + j] &= (2 * j + 8 < keep ? 0xFFFFu : 0u) | (2 * j + 9 < keep ? 0xFFFF0000u : 0u);
                    }
                } else {
                    const int keep = ctx - (t * BN + unit * 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = j < keep ? x[j] : 0u;
                }
                *p = x;
            }
        }
    };
    if (!kExact) {                                              // channels the cache does not have: zero keys
        const int have = (D >> 3) * 1024;
        for (int i = have + tid * 16; i < kTile; i += 256 * 16) {
            *reinterpret_cast<u32x4*>(lds + i) = u32x4{0, 0, 0, 0};
            *reinterpret_cast<u32x4*>(lds + 2 * kTile + i) = u32x4{0, 0, 0, 0};
        }
    }

    const float unit_scale = kBf16 ? a.scale * kLog2e : a.scale;   // bf16 takes its weights as powers of two
    float m = -INFINITY, lsum = 0.f;
    f32x16 o[DT / 32];
#pragma unroll
    for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mb][i] = 0.f;

    Pages pg;
    pages_of(0, pg);
    request(0, 0, pg);
    pages_of(min(1, n_tiles - 1), pg);
    AG_WAIT_VMCNT(0);
    scrub_v(0, 0);
    __syncthreads();

#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) {
        if (t + 1 < n_tiles) {
            request(t + 1, (t + 1) & 1, pg);
            pages_of(min(t + 2, n_tiles - 1), pg);
        }
        if (t < wave_tiles) {
            const unsigned char* kb = lds + (t & 1) * 2 * kTile + hi * (kBf16 ? 1024 : 512) + n * 16;
            const unsigned char* vb = lds + (t & 1) * 2 * kTile + kTile + hi * DT * 16 + n * 16;
            f32x16 sc[2];
#pragma unroll
            for (int i = 0; i < 16; ++i) { sc[0][i] = 0.f; sc[1][i] = 0.f; }
            float x[kScores];
            if constexpr (kBf16) {
                with_operands<DT / 8>([&](int i) { return kb + (i & 1) * 512 + (i >> 1) * 2048; }, [&](int i, u32x4 k) {
                    sc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, qf[i >> 1]), sc[i & 1], 0, 0, 0);
                });
#pragma unroll
                for (int i = 0; i < 32; ++i) x[i] = sc[i >> 4][i & 15];
            } else {
                with_operands<DT / 8>([&](int i) { return kb + i * 1024; }, [&](int i, u32x4 k) {
                    const f32x4 kf = __builtin_bit_cast(f32x4, k), q4 = __builtin_bit_cast(f32x4, qf[i]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], q4[e], sc[e & 1], 0, 0, 0);
                });
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = sc[0][i] + sc[1][i];
            }
            if (t >= first_masked) {                            // the tile straddles this wave's diagonal
#pragma unroll
                for (int i = 0; i < kScores; ++i) {
                    const int key = t * BN + (i >> 2) * 8 + hi * 4 + (i & 3);
                    x[i] = key <= qpos ? x[i] : -INFINITY;
                }
            }
            float mx = x[0];
#pragma unroll
            for (int i = 1; i < kScores; ++i) mx = fmaxf(mx, x[i]);
            mx *= unit_scale;                                   // scale > 0: max and scaling commute
            // m is shared by the two lanes of a column: if either lane's own maximum outgrew it, combine them
            if (__builtin_amdgcn_ballot_w64(mx > m + kSlack) != 0) {
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float m_new = fmaxf(m, mx);
                const float alpha = m_new == -INFINITY ? 1.f : kBf16 ? __builtin_amdgcn_exp2f(m - m_new) : expf(m - m_new);
                lsum *= alpha;
#pragma unroll
                for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[mb][i] *= alpha;
                m = m_new;
            }
            const float m_ref = m == -INFINITY ? 0.f : m;
            float psum = 0.f;
#pragma unroll
            for (int i = 0; i < kScores; ++i) {
                const float e = fmaf(x[i], unit_scale, -m_ref);
                x[i] = kBf16 ? __builtin_amdgcn_exp2f(e) : expf(e);
                psum += x[i];
            }
            lsum += psum;
            constexpr int kMb = DT / 32;
            if constexpr (kBf16) {
                Terms p[4];                                     // the weights, in k-step order
#pragma unroll
                for (int i = 0; i < 16; ++i) p[i >> 2].set_pair(i & 3, x[2 * i], x[2 * i + 1]);
                with_operands<4 * kMb>([&](int i) { return vb + (i / kMb) * 2 * DT * 16 + (i % kMb) * 512; }, [&](int i, u32x4 v) {
                    const bf16x8 vv = __builtin_bit_cast(bf16x8, v);
                    o[i % kMb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, __builtin_bit_cast(bf16x8, p[i / kMb].l), o[i % kMb], 0, 0, 0);
                    o[i % kMb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, __builtin_bit_cast(bf16x8, p[i / kMb].m), o[i % kMb], 0, 0, 0);
                    o[i % kMb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, __builtin_bit_cast(bf16x8, p[i / kMb].h), o[i % kMb], 0, 0, 0);
                });
            } else {
                with_operands<4 * kMb>([&](int i) { return vb + (i / kMb) * 2 * DT * 16 + (i % kMb) * 512; }, [&](int i, u32x4 v) {
                    const f32x4 vv = __builtin_bit_cast(f32x4, v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[i % kMb] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[e], x[(i / kMb) * 4 + e], o[i % kMb], 0, 0, 0);
                });
            }
        }
        AG_WAIT_VMCNT(0);                                       // this wave's part of tile t + 1 has landed
        if (t + 1 < n_tiles) scrub_v(t + 1, (t + 1) & 1);
        __syncthreads();
    }

    // o[mb][q4 * 4 + e] is O^T[channel mb * 32 + q4 * 8 + hi * 4 + e][column n]
    lsum += __shfl_xor(lsum, 32);
    const float inv = 1.0f / lsum;
    float trouble = general::trouble_of(inv);
#pragma unroll
    for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) trouble = general::trouble_of(o[mb][i], trouble);
    uint64_t again = __builtin_amdgcn_ballot_w64(n < cols_w && !(trouble == 0.f));
    again = (again | (again >> 32)) & 0xFFFFFFFFu;              // bit c: column c of this wave
    if (n < cols_w && !((again >> n) & 1)) {
        E* out = (E*)a.out + row * D + hi * 4;
#pragma unroll
        for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int d = mb * 32 + q4 * 8;
                if (!kExact && d >= D) break;
                if constexpr (kBf16) {
                    bf16x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = (__bf16)(o[mb][q4 * 4 + e] * inv);
                    *reinterpret_cast<bf16x4*>(out + d) = y;
                } else {
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = o[mb][q4 * 4 + e] * inv;
                    *reinterpret_cast<f32x4*>(out + d) = y;
                }
            }
    }
    general::attend_rows_again<E, rows_again(DT), DT / 64>(a, again, row, qpos, s, g, reinterpret_cast<float*>(lds) + rows_again(DT) * DT * wu);       // (all are past the last tile)
}

// sum_s ceil(N_s G / 128) <= total G / 128 + batch, and no session has more than ceil(max_new G / 128)
int64_t tiles_bound(const AttnArgs& a)
{
    const int64_t G = a.hq / a.c.hkv;
    return std::min<int64_t>((int64_t)a.total_rows * G / kColumns + a.batch, (int64_t)a.batch * ((a.max_new * G + kColumns - 1) / kColumns));
}

template <typename E, int DT, bool kExact>
ag_status launch_kernel(const AttnArgs& a, hipStream_t st)
{
    constexpr int lds = 512 * DT;
    if constexpr (lds > 64 * 1024) {
        static std::atomic<uint64_t> told{0};
        ag_status e = allow_dynamic_lds((const void*)prefill_any_kernel<E, DT, kExact>, lds, told);
        if (e) return e;
    }
    const Deal deal = deal_of(a, tiles_bound(a), stream_cus(st) * (DT > 128 ? 1 : 2) / 8);
    prof_before(st);
    hipLaunchKernelGGL((prefill_any_kernel<E, DT, kExact>), dim3((unsigned)workgroups_of(deal)), dim3(256), lds, st, a, deal);
    prof_after(st);
    return hip_check(hipGetLastError(), "prefill launch");
}

template <typename E>
ag_status launch_for_dim(const AttnArgs& a, hipStream_t st)
{
    if constexpr (sizeof(E) == 2) {                 // (fp32 at 64 and 128, and bf16 at 128, never come here)
        if (a.c.d == 64) return launch_kernel<E, 64, true>(a, st);
    }
    if (a.c.d <= 64) return launch_kernel<E, 64, false>(a, st);
    if (a.c.d <= 128) return launch_kernel<E, 128, false>(a, st);
    return a.c.d == 256 ? launch_kernel<E, 256, true>(a, st) : launch_kernel<E, 256, false>(a, st);
}

}  // namespace

// Pages below 16 tokens store V without the 8-key chunks these loads rely on, and pointers off 16 bytes rule out
// 16-byte accesses: both stay with the general kernel, as does a batch whose tile list does not fit one launch.
bool prefill_any_supported(const AttnArgs& a)
{
    return a.c.ps >= 16 && (((uintptr_t)a.q | (uintptr_t)a.out | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 == 0) &&
           a.c.hkv * tiles_bound(a) + kDealtPast <= 0x7fffffff && (int64_t)a.total_rows * (a.hq / a.c.hkv) <= 0x7fffffff;
}

ag_status launch_prefill_any(const AttnArgs& a, hipStream_t st)
{
    if (prefill_mfma_lo_supported(a)) return launch_prefill_mfma_lo(a, st);
    if (prefill_split_preferred(a, false, st)) return launch_prefill_split(a, false, st);
    if (prefill_f32_supported(a)) return launch_prefill_f32(a, st);
    return a.c.dtype == AG_BF16 ? launch_for_dim<__bf16>(a, st) : launch_for_dim<float>(a, st);
}

}  // namespace ag
