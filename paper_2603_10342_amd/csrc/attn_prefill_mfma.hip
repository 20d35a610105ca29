// Cold and resume prefill over a paged KV cache, bf16, head_dim 64 or 128, pages of 16 tokens or more
// (paper Sec. I and Sec. II-A: a cold prefill is full causal attention over
// the prompt; a resume prefill appends a chunk to a cached context, so row i
// of a session with P cached tokens sees keys 0 .. P + i.  Cold is P = 0.)
//
// A dense contraction, bound by the matrix cores: 4 * D flop per visible
// (query, key) pair and head.  One workgroup of NW waves (4 or 8) owns 32 * NW
// columns of one (session, KV head): a column is a (token, query head of the
// group) pair, numbered token * G + head, so that any group size and chunk
// length fills its tiles and all heads of the group share K and V; each wave
// owns 32 columns and keeps their Q in registers.  Keys and
// values are taken 64 at a time and staged through LDS by direct
// global-to-LDS loads:
//
//   S^T[key][query] = K[key][:] . Q[query][:]      2 x D/16 MFMA 32x32x16
//   softmax weights per query column (reference m, running sum l, exp2)
//   O^T[d][query]  += V^T[d][key] . P^T[key][query]  D/32 x 4 MFMA 32x32x16
//
// Computing the transposed score tile puts one query in one lane (plus its
// partner lane + 32), so the row max / sum need a single cross-lane step,
// and the 8 scores a lane holds for one k-step of the second product are
// already its B operand: P never leaves registers.  The pools' page layouts
// are the LDS tile layouts (K chunk-major, V transposed in 8-key chunks in the
// slot order the score tile produces), so a tile is copied as contiguous runs,
// 16-byte operand reads are conflict free and every operand address is the
// lane's base plus a constant.
//
// The per-element softmax work on the vector ALUs is about as long as the
// matrix work (one exp per 512 flop), so iteration t of a wave interleaves,
// instruction by instruction, O += V(t-1).P(t-1) (matrix) with
// P(t) = exp2(S(t) - m) (vector), after S(t) = K(t).Q^T.  m is a reference,
// not the running maximum: the common case takes the weights under the current
// m and only checks afterwards that none came out large; a wave's first tile
// and a failed check take an ordered path that finds the row maxima, rescales
// O and l when a maximum outgrew m by more than 2^8, and recomputes the weights.
// Tiles wholly above a wave's rows are skipped; the tiles on the diagonal are
// masked before the weights are taken.
//
// KV heads are dealt to the XCDs (tile_list.h), and a head's tiles are listed
// session-major, longest context first: the workgroups resident together read
// few sessions' K/V for one KV head, which then stays in that XCD's L2.  The grid lists the batch's real
// tiles only (each workgroup finds its tile from the chunk lengths): empty
// workgroups are not free, the dispatcher takes as long over them as over
// the others.
#include <algorithm>
#include <atomic>

#include "ag_internal.h"
#include "attn_general_row.h"
#include "attn_tile32.h"
#include "lds_dma.h"
#include "tile_list.h"

namespace ag {

namespace {

using namespace tile32;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// K stages: 3 (K(t+2) is requested while K(t) is used); V stages: 2 (V(t) requested while V(t-1) is used; a third
// measured no faster).  At head_dim 128 that is 80 KiB: two 4-wave workgroups or one 8-wave workgroup per CU.
constexpr int kVStages = 2;
// The 8-wave form also keeps two windows of 64 page ids (16 key tiles each) of the session's block-table row in
// LDS, see the kernel; the 4-wave form at head_dim 128 has no room for them (two workgroups of 80 KiB fill a CU's LDS).
constexpr int kIdWindow = 64;
constexpr bool ids_in_lds(int nw) { return nw == 8; }
constexpr int lds_bytes(int nw, int dt) { return (kKStages + kVStages) * tile_bytes(dt) + (ids_in_lds(nw) ? 2 * kIdWindow * 4 : 0); }

// NW waves per workgroup (4 or 8), 32 columns each.  Eight waves halve the K/V bytes moved per flop (a tile
// is shared by twice the columns) at the price of coarser query tiles.  kLo: weights as three bf16 terms
// (attn_tile32.h); the bf16 / 128 / 16 shape runs without.  kPage16: pages of 16 tokens, whose groups need no place
// inside the page.
// kHalves: two sets of NW waves take every other key tile of the same columns, see prefill_halves_kernel.
template <int NW, int DT, bool kLo, bool kPage16, int kHalves>
__device__ __forceinline__ void attend_tile(const AttnArgs& a, const Deal& deal)
{
    constexpr int kCols = 32 * NW;          // columns per workgroup
    constexpr int kTile = tile_bytes(DT);
    constexpr int kPer = DT / 8 / NW;       // direct-load instructions per wave for a K tile, and for a V tile
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    // ---- which (KV head, session, query tile) ----
    const int hkv = a.c.hkv, hq = a.hq, G = hq / hkv;
    // Work order: KV head, then session, then query tile (longest first).
    // The grid holds `tiles_max` tiles per KV head, a host-side bound on sum_s ceil(N_s G / kCols); which (session,
    // tile) the workgroup's tile index means follows from the lengths, which every wave scans for itself.
    // A grid of batch x ceil(max_new G / kCols) tiles would be mostly empty
    // workgroups when chunk lengths differ much, and launching a workgroup of this size takes the dispatcher of
    // an XCD most of a microsecond, whether it has work or not.
    int g, j;
    if (!place_of(deal, hkv, g, j)) return;
    int s = -1, qt = 0, N = 0, P = 0, row0 = 0;
    find_tile<kCols>(a, j, G, s, qt, N, P, row0);
    if (s < 0) return;                              // beyond the batch's tiles
    const int ctx = P + N;
    const int tid = threadIdx.x, w = kHalves == 1 ? tid >> 6 : (tid >> 6) & (NW - 1), lane = tid & 63;
    const int wu = __builtin_amdgcn_readfirstlane(w);           // the same value, known to be uniform: used only
                                                                 // where a scalar is required (page ids, M0)
    const int half = kHalves == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / NW;
    auto tile = [&](int t) { return kHalves == 1 ? t : kHalves * t + half; };      // the key tile of iteration t
    const int n = lane & 31, hi = lane >> 5;
    const __bf16* kpool = (const __bf16*)a.c.k;
    const __bf16* vpool = (const __bf16*)a.c.v;
    // the block table is read-only for the kernel's lifetime: reading it through the constant address space
    // lets the (uniform) page-id loads be scalar loads, which use their own counter
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    const cptr_t bt = (cptr_t)(uintptr_t)(a.bt + (int64_t)s * a.max_pages);
    // 16-token groups: group i of the context is group i & gmask of logical page i >> gshift
    const int last_grp = (ctx - 1) >> 4;
    const int gshift = kPage16 ? 0 : a.c.ps_shift - 4, gmask = kPage16 ? 0 : (1 << gshift) - 1;
    const int64_t block = kPage16 ? DT * 16 : (int64_t)DT * a.c.ps;            // elements of one (page, head)
    const int k_stride = kPage16 ? 256 : a.c.ps * 16;                          // bytes between a K page's chunks

    // ---- tile requests: direct global-to-LDS loads, kPer + kPer wave-wide instructions per wave and tile ----
    unsigned char* const k_lds = lds + half * ((kKStages + kVStages) * kTile);     // K of iteration t lives at k_lds + (t % 3) * kTile
    unsigned char* const v_lds = k_lds + kKStages * kTile;                         // V at v_lds + (t % 2) * kTile
    const int kgrp = lane >> 4, kslot = lane & 15;          // K: lane = key of the tile (group, slot)
    const int kmask[4] = {kgrp == 0 ? -1 : 0, kgrp == 1 ? -1 : 0, kgrp == 2 ? -1 : 0, kgrp == 3 ? -1 : 0};

    // Physical pages of a tile's groups.  Scalar form (the prologue, and the 4-wave kernel throughout): scalar loads (the
    // index is uniform), fetched one iteration before the tile's data is requested.  A scalar load in flight
    // costs more than its latency, though: it shares a counter with the LDS operand reads and returns out of
    // order, so while one is pending every wait for an operand becomes a wait for everything.  The 8-wave
    // kernel therefore keeps the ids in LDS: wave 0 brings the session's groups in windows of 64
    // (16 key tiles) by one direct load each, two windows resident, and every lane reads the id it needs
    // (its own group's of the K tile, the wave's group's of the V tile) with an ordinary LDS read.
    constexpr bool kLdsIds = ids_in_lds(NW);
    static_assert(!kLdsIds || kHalves == 1, "two sets of waves leave no room for page ids");
    struct Pages { int k; int v; };                            // k: the page of this LANE's group of the K tile; v: of the wave's group of the V tile
    const int v_grp = (wu * 4) / NW;                           // group of a V tile this wave brings in (a group's two 8-key chunks)
    auto id_of = [&](int grp) { return bt[min(grp, last_grp) >> gshift]; };
    auto pages_scalar = [&](int tk, int tv, Pages& pg) {
        int pid[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pid[i] = id_of(tk * 4 + i);
        // this lane's page among the four (uniform) ids, by masks: a chain of ?: here compiles to branches
        pg.k = (pid[0] & kmask[0]) | (pid[1] & kmask[1]) | (pid[2] & kmask[2]) | (pid[3] & kmask[3]);
        pg.v = id_of(tv * 4 + v_grp);
    };
    const int32_t* const id_lds = reinterpret_cast<const int32_t*>(lds + (kKStages + kVStages) * kTile);
    // window w = groups [64 w, 64 w + 64), clamped to the session's last group, into slot w & 1
    auto refill_ids = [&](int win) {
        const int grp = min(win * kIdWindow + lane, last_grp);
        load_dword_to_lds(a.bt + (int64_t)s * a.max_pages + (grp >> gshift), lds_address(id_lds) + (win & 1) * (kIdWindow * 4));
    };
    auto pages_of = [&](int tk, int tv, Pages& pg) {
        if constexpr (kLdsIds) {
            pg.k = id_lds[(tk * 4 + kgrp) & (2 * kIdWindow - 1)];
            pg.v = id_lds[(tv * 4 + v_grp) & (2 * kIdWindow - 1)];       // uniform; made scalar where it is used
        } else {
            pages_scalar(tk, tv, pg);
        }
    };
    // K(t): instruction i of wave w moves chunk c = kPer*w + i of all 64 keys: four 256-byte runs, one per group.
    // (t beyond the last tile repeats it: tk is the tile that is read, stage_t the one whose place it takes.)
    auto request_k = [&](int tk, int stage_t, int mine) {
        const unsigned char* src = (const unsigned char*)kpool + ((int64_t)mine * hkv + g) * (block * 2) + (int64_t)(wu * kPer) * k_stride + kslot * 16;
        if (!kPage16) src += (min(tk * 4 + kgrp, last_grp) & gmask) * 256;
        const unsigned dst = lds_address(k_lds) + (stage_t % kKStages) * kTile + (wu * kPer) * 1024;
#pragma unroll
        for (int i = 0; i < kPer; ++i) load_to_lds(src + (int64_t)i * k_stride, dst + i * 1024);
    };
    // V(tv): a group's [half][channel][8 keys] layout is the LDS layout, so a V tile is DT/8 runs of 1 KiB;
    // wave w moves runs kPer*w .. kPer*w + kPer - 1, all of group v_grp.
    constexpr int kRunsPerGroup = DT / 32, kRunsPerHalf = DT / 64;
    auto request_v = [&](int tv, int stage, int pid_any_lane) {
        const int pid = __builtin_amdgcn_readfirstlane(pid_any_lane);
        const unsigned char* src = (const unsigned char*)vpool + ((int64_t)pid * hkv + g) * (block * 2) +
                                   ((wu * kPer) % kRunsPerGroup) * 1024 + lane * 16;
        if (!kPage16) src += (int64_t)(min(tv * 4 + v_grp, last_grp) & gmask) * (DT * 32);
        const unsigned dst = lds_address(v_lds) + stage * kTile + (wu * kPer) * 1024;
#pragma unroll
        for (int i = 0; i < kPer; ++i) load_to_lds(src + i * 1024, dst + i * 1024);
    };
    // Slots behind the session's last token may contain anything (NaN included) and would poison
    // the value product even under a zero weight: once V(tv) has landed, zero them in LDS.
    auto scrub_v = [&](int stage, int tv) {
        const int keep = ctx - (tv * BN + v_grp * 16);          // slots < keep of this wave's group hold tokens
        if (keep < 16) {                                        // uniform over the wave
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int half = ((wu * kPer) % kRunsPerGroup + i) / kRunsPerHalf;
                u32x4* p = reinterpret_cast<u32x4*>(v_lds + stage * kTile + (wu * kPer + i) * 1024 + lane * 16);
                *p = keep_quads(*p, keep - half * 4, keep - 8 - half * 4);
            }
        }
    };

    // ---- prologue: K(0), K(1) (and the first window of page ids) are on their way before anything else is worked out: what
    // follows - the columns, Q - takes longer than their addresses (a long cold prefill: 1 %) ----
    Pages pg;
    if constexpr (kLdsIds) {
        if (wu == 0) refill_ids(0);
    }
    pages_scalar(tile(0), 0, pg);
    request_k(tile(0), 0, pg.k);
    pages_scalar(tile(1), 0, pg);                    // (beyond a short context's last group the ids repeat: read, never used)
    request_k(tile(1), 1, pg.k);

    const int col0 = qt * kCols;
    const int cols = min(N * G - col0, kCols);                  // valid columns of this workgroup
    const Columns columns(col0, G);

    const int cols_w = max(0, min(32, cols - 32 * wu));         // valid columns of this wave
    const int col = min(32 * wu + n, cols - 1);                 // columns beyond the tile repeat the last one
    const int token = columns.token(col);
    const int64_t base_row = (int64_t)row0 * hq + (int64_t)g * G;             // row (token 0, head 0) of Q and O
    const unsigned my_row = (unsigned)token * (unsigned)hq + (unsigned)columns.head(col, token);      // this lane's, from there

    const int n_tiles = (P + columns.token(cols - 1)) / BN + 1;               // tiles the workgroup stages
    const int wave_tiles = cols_w > 0 ? (P + columns.token(32 * wu + cols_w - 1)) / BN + 1 : 0;      // tiles this wave uses
    const int first_masked = (P + columns.token(32 * wu) + 1) / BN;   // first tile holding a key this wave's first column may not see

    // ---- Q^T as B operand: column n, k-step ks covers channels ks*16 + hi*8 .. +7 ----
    bf16x8 qf[DT / 16];
    {
        const __bf16* qp = (const __bf16*)a.q + (base_row + my_row) * DT + hi * 8;
#pragma unroll
        for (int ks = 0; ks < DT / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
    }

    const float sl2 = a.scale * kLog2e;
    const int qpos = P + token;                     // logical position of this lane's query
    float m = -INFINITY, lsum = 0.f;
    f32x16 o[DT / 32];
#pragma unroll
    for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mb][i] = 0.f;

    const unsigned char* const k_lane = k_lds + n * 16 + hi * 1024;
    const unsigned char* const v_lane = v_lds + n * 16 + hi * (DT * 16);

    pages_scalar(min(tile(2), n_tiles - 1), min(tile(0), n_tiles - 1), pg);        // what iteration 0 requests: V(0) and K(2)
    AG_WAIT_VMCNT(0);
    __syncthreads();
    f32x16 sc[2];
    Weights<kLo> pa, pb;

    // Iteration t of a wave: S(t) from K(t) (matrix); then P(t) = exp2(S(t) - m) (vector) side by side with
    // O += V(t-1).P(t-1) (matrix).  At its start it requests V(t) and then K(t+2); at its end it waits until only
    // its own K(t+2) loads are outstanding, i.e. V(t) and K(t+1) have landed.
    // Requests are unconditional (past the last tile they repeat it into a buffer nobody reads), so the loop body has one
    // shape.  Every wave runs all n_tiles + 1 iterations (the barriers are workgroup-wide); the pieces a wave
    // does not need are skipped.
    auto iter = [&](int t, Weights<kLo>& p_prev, Weights<kLo>& p_cur) {
        const int tv = min(tile(t), n_tiles - 1);    // the V tile that must have landed when this iteration ends
        if constexpr (kLdsIds) {
            // The window holding tile t + 4 comes in one iteration before its first id is read (iteration t + 1
            // reads those of K(t + 4)); issued ahead of this iteration's tile requests, it has landed when wave 0
            // passes the wait at the end of the iteration, and the barrier there shows it to the other waves.
            // The slot it replaces holds the window two back, which nothing reads any more.
            if (wu == 0 && ((t + 4) & 15) == 0) refill_ids((t + 4) >> 4);
        }
        request_v(tv, t % kVStages, pg.v);
        request_k(min(tile(t + 2), n_tiles - 1), t + 2, pg.k);
        Pages nxt;                                    // ids for the next iteration's requests
        pages_of(min(tile(t + 3), n_tiles - 1), min(tile(t + 1), n_tiles - 1), nxt);
        const bool do_sm = tile(t) < wave_tiles, do_pv = t >= 1 && tile(t - 1) < wave_tiles;
        const unsigned char* kb = k_lane + (t % kKStages) * kTile;
        const unsigned char* vb = v_lane + ((t + kVStages - 1) % kVStages) * kTile;   // V(t-1)
        if (do_sm) {
            qk_tile<DT>(kb, qf, sc);
            if (tile(t) >= first_masked) {           // the tile straddles this wave's diagonal
                const int kbase = tile(t) * BN + hi * 4;
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int key = kbase + b * 32 + (i >> 2) * 8 + (i & 3);
                        sc[b][i] = key <= qpos ? sc[b][i] : -INFINITY;
                    }
            }
        }
        softmax_and_value_product<DT, kLo>(do_sm, do_pv, vb, sc, sl2, m, lsum, p_prev, p_cur, o);
        AG_WAIT_VMCNT(kPer);
        scrub_v(t % kVStages, tv);
        pg = nxt;
        __syncthreads();
    };

#pragma unroll 1
    for (int t = 0; t <= (n_tiles + kHalves - 1) / kHalves; t += 2) {
        iter(t, pb, pa);
        if (t + 1 <= (n_tiles + kHalves - 1) / kHalves) iter(t + 1, pa, pb);
    }

    // ---- normalise, transpose through LDS, store rows contiguously ----
    AG_WAIT_VMCNT(0);                                // the last (redundant) tile requests still write to LDS
    __syncthreads();
    if constexpr (kHalves == 2) {                    // the second half's sums, lane by lane
        f32x4* const part = reinterpret_cast<f32x4*>(lds + w * (DT * 128)) + lane;
        float* const ml = reinterpret_cast<float*>(lds + NW * (DT * 128)) + w * 128 + lane;
        if (half == 1) {
#pragma unroll
            for (int i = 0; i < DT / 8; ++i)
                part[i * 64] = f32x4{o[i >> 2][(i & 3) * 4], o[i >> 2][(i & 3) * 4 + 1], o[i >> 2][(i & 3) * 4 + 2], o[i >> 2][(i & 3) * 4 + 3]};
            ml[0] = m;
            ml[64] = lsum;
        }
        __syncthreads();
        if (half == 1) return;
        const float m1 = ml[0], top = fmaxf(m, m1);
        const float f0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - top), f1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - top);
        lsum = lsum * f0 + ml[64] * f1;
#pragma unroll
        for (int i = 0; i < DT / 8; ++i) {
            const f32x4 x = part[i * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[i >> 2][(i & 3) * 4 + e] = o[i >> 2][(i & 3) * 4 + e] * f0 + x[e] * f1;
        }
    }
    lsum += __shfl_xor(lsum, 32);
    const float inv = 1.0f / lsum;
    constexpr int kChunks = DT / 8;                 // 16-byte pieces of a row
    uint64_t again = 0;
    if constexpr (kLo) {
        float trouble = general::trouble_of(inv);
#pragma unroll
        for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) trouble = general::trouble_of(o[mb][i], trouble);
        again = __builtin_amdgcn_ballot_w64(n < cols_w && !(trouble == 0.f));
    }
    unsigned char* ob = lds + w * (32 * DT * 2 * kHalves);      // (where this wave read its sums)  this wave's [32 columns][DT ch] bf16, rows XOR-swizzled
#pragma unroll
    for (int mb = 0; mb < DT / 32; ++mb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            bf16x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (__bf16)(o[mb][q4 * 4 + e] * inv);
            const int d = mb * 32 + q4 * 8 + hi * 4;            // 4 consecutive channels
            const int chunk = d >> 3;
            *reinterpret_cast<bf16x4*>(ob + n * (DT * 2) + ((chunk ^ (n & (kChunks - 1))) << 4) + (d & 7) * 2) = x;
        }
    __syncthreads();
    {
        const int c = lane % kChunks;
        __bf16* outp = (__bf16*)a.out + base_row * DT + c * 8;
#pragma unroll
        for (int k = 0; k < kChunks / 2; ++k) {
            const int r = lane / kChunks + (64 / kChunks) * k;              // column of the wave: lane r knows its row
            const unsigned row = (unsigned)__shfl((int)my_row, r);
            if (r < cols_w) {
                const u32x4 x = *reinterpret_cast<const u32x4*>(ob + r * (DT * 2) + ((c ^ (r & (kChunks - 1))) << 4));
                *reinterpret_cast<u32x4*>(outp + (int64_t)row * DT) = x;
            }
        }
    }
    if constexpr (kLo) {
        again = (again | (again >> 32)) & 0xFFFFFFFFu;          // bit c: column c of this wave
        general::attend_rows_again<__bf16, 4, DT / 64>(a, again, (int64_t)base_row + (unsigned)my_row, qpos, s, g, reinterpret_cast<float*>(ob));
    }
}

template <int NW, int DT, bool kLo, bool kPage16>
__global__ __launch_bounds__(64 * NW, 2) void prefill_mfma_kernel(AttnArgs a, Deal deal) { attend_tile<NW, DT, kLo, kPage16, 1>(a, deal); }

// Few workgroups on long contexts: a launch is as long as its longest chain of key tiles, one wave a SIMD.  Here two sets of four
// waves take every other tile of the same 128 columns, with key and value stages of their own, and their sums meet in LDS at the
// end; a CU holds one such workgroup instead of two.  Which batches: launch_tiles().
template <int DT, bool kLo, bool kPage16>
__global__ __launch_bounds__(512, 2) void prefill_halves_kernel(AttnArgs a, Deal deal) { attend_tile<4, DT, kLo, kPage16, 2>(a, deal); }

}  // namespace

static bool aligned16(const AttnArgs& a)
{
    return ((uintptr_t)a.q | (uintptr_t)a.out | (uintptr_t)a.c.k | (uintptr_t)a.c.v) % 16 == 0;
}

// the bf16 / 128 / 16 shape, whose weights are rounded to bf16
bool prefill_mfma_supported(const AttnArgs& a)
{
    return a.c.dtype == AG_BF16 && a.c.d == 128 && a.c.ps == 16 && aligned16(a);
}

// sum_s ceil(N_s G / cols) <= total G / cols + batch, and no session has more than ceil(max_new G / cols)
static int64_t tiles_bound(const AttnArgs& a, int cols)
{
    const int64_t G = a.hq / a.c.hkv;
    return std::min<int64_t>((int64_t)a.total_rows * G / cols + a.batch, (int64_t)a.batch * ((a.max_new * G + cols - 1) / cols));
}

// Other bf16 batches that take this kernel, with weights in 32 bits: head_dim 128 (32-token pages, append included, the general tiles -> this one:
// eight chunks of 40..500 rows on 500..4000 tokens 210 -> 199 us, eight prompts of 2048 528 -> 523), and head_dim 64 when
// contexts are over twice the chunks.  There the interleaved softmax shortens a workgroup's chain of tiles, and the longer
// start of its pipeline and the lower occupancy lengthen a launch of many workgroups.  64-token pages, general tiles -> this
// one: the same chunks 144 -> 129 us (a launch as long as its longest chain); 32 chunks of 300 rows on 150 tokens 89 ->
// 97, on 300 114 -> 118, on 600 161 -> 166, on 2000 381 -> 387; eight of 2000 on 0, 500, 1000 336 -> 336, 445 -> 444, 567
// -> 563, on 1900, 2100, 3000 787 -> 778, 832 -> 825, 1060 -> 1051.  Around the line the two are within 3 %.
bool prefill_mfma_lo_supported(const AttnArgs& a)
{
    return a.c.dtype == AG_BF16 && (a.c.d == 128 || (a.c.d == 64 && a.max_ctx > 2 * (int64_t)a.max_new)) && a.c.ps >= 16 && aligned16(a) &&
           a.c.hkv * tiles_bound(a, 128) + kDealtPast <= 0x7fffffff && (int64_t)a.total_rows * (a.hq / a.c.hkv) <= 0x7fffffff;
}

template <int NW, int DT, bool kLo, bool kPage16>
static ag_status launch_prefill_nw(const AttnArgs& a, hipStream_t st)
{
    constexpr int lds = lds_bytes(NW, DT);
    if constexpr (lds > 64 * 1024) {
        static std::atomic<uint64_t> told{0};
        ag_status e = allow_dynamic_lds((const void*)prefill_mfma_kernel<NW, DT, kLo, kPage16>, lds, told);
        if (e) return e;
    }
    if (a.c.hkv * tiles_bound(a, 32 * NW) + kDealtPast > 0x7fffffff) { set_error("too many query tiles for one launch"); return AG_ERR_INVALID_ARG; }
    const Deal deal = deal_of(a, tiles_bound(a, 32 * NW), stream_cus(st) * (8 / NW) / 8);
    prof_before(st);
    hipLaunchKernelGGL((prefill_mfma_kernel<NW, DT, kLo, kPage16>), dim3((unsigned)workgroups_of(deal)), dim3(64 * NW), lds, st, a,
                       deal);
    prof_after(st);
    return hip_check(hipGetLastError(), "prefill launch");
}

template <int DT, bool kLo, bool kPage16>
static ag_status launch_prefill_halves(const AttnArgs& a, hipStream_t st)
{
    constexpr int lds = 2 * lds_bytes(4, DT);
    static std::atomic<uint64_t> told{0};
    ag_status e = allow_dynamic_lds((const void*)prefill_halves_kernel<DT, kLo, kPage16>, lds, told);
    if (e) return e;
    if (a.c.hkv * tiles_bound(a, 128) + kDealtPast > 0x7fffffff) { set_error("too many query tiles for one launch"); return AG_ERR_INVALID_ARG; }
    const Deal deal = deal_of(a, tiles_bound(a, 128), stream_cus(st) / 8);
    prof_before(st);
    hipLaunchKernelGGL((prefill_halves_kernel<DT, kLo, kPage16>), dim3((unsigned)workgroups_of(deal)), dim3(512), lds, st, a, deal);
    prof_after(st);
    return hip_check(hipGetLastError(), "prefill launch");
}

// lo: weights in 32 bits (see kLo)
static ag_status launch_tiles(const AttnArgs& a, bool lo, hipStream_t st)
{
    if (prefill_split_preferred(a, !lo, st)) return launch_prefill_split(a, !lo, st);
    // 256-column workgroups (a K/V tile then feeds twice the columns) when chunks are long enough to fill them and the batch
    // spreads over at least 5/8 of the CUs.  128-column workgroups keep short, ragged chunks efficient and spread small batches (one
    // chunk on 6000 tokens, whole call: 600 rows 152 -> 126 us, 1000 rows 167 -> 139).  They also end a launch better: 256 columns
    // are one workgroup a CU, whose start (4 us) and end nothing else hides and of which a last one a CU is a long one, so that
    // two workgroups of 128 columns a CU win on contexts up to 1536 unless all of the larger ones run at once, however many there
    // are, and on longer ones while the larger ones come to few a CU - unless all of them run at once and are alike, so that there
    // is nothing to even out: chunks of one length, short beside their contexts (a tile's keys grow over a chunk).
    // Graph replay, append included, 256 -> 128 columns, us (of the larger a CU).  Rounded weights: four prompts of 600 (1.3) 37.8 ->
    // 32.5, seven of 700..912 at 16 / 2 heads (1.4) 52 -> 47, one of 2048 (1) 62.5 -> 58.2, three of 700 on 2000 (1.03) 127 -> 118, 16 of
    // 1500 (12) 401 -> 386, 64 of 600, 1000, 1500 (20, 32, 48) 382 -> 364, 856 -> 803, 1568 -> 1510; but two of 1000 (1) 38.9 -> 40.3,
    // two of 1000 on 2000 (1) 93 -> 97, four of 512 on 3000 (1) 112 -> 116, six of 1024 on 4000 at 8 / 2 (0.75) 131 -> 139, eight of
    // 512..600 on 2000..4000 (2.2) 261 -> 268.  Weights in 32 bits: one of 2048 (1) 101 -> 85, three of 700 on 2000 (1.03) 218 -> 189, 64 of
    // 1000, 1500 (32, 48) 1316 -> 1211, 2567 -> 2392; but two of 600 on 6000 (0.62) 283 -> 310, one of 3000 on 3000 at 16 / 2 (0.73) 264 -> 281, six of 1024 on 4000 at 8 / 2
    // (0.75) 229 -> 251, two of 1000 on 2000 (1) 160 -> 170, four of 2048 (4) 265 -> 274.  Over 1540 drawn batches of 0.6 to 3.2 a CU, also
    // on 64 and 160 CUs, this line is 1.04 times faster than 256 columns from 5/8 of the CUs on; it is over 3 % slower at 75, of which 58
    // are of more than one round, where the order in which unlike workgroups come to a CU decides.
    const int64_t cus = stream_cus(st), large = a.c.hkv * tiles_bound(a, 256);         // workgroups of 256 columns
    const bool ragged = 5 * (int64_t)a.total_rows < 4 * (int64_t)a.batch * a.max_new;
    const int64_t rows = a.max_new, ctx = a.max_ctx;
    const bool alike = !ragged && (lo ? 3 * rows <= ctx || (10 * large > 7 * cus && 5 * rows <= 4 * ctx) : 5 * rows <= 2 * ctx);
    const bool pays = large <= cus ? a.max_ctx <= 1536 || alike : a.max_ctx > 1536 && 4 * large >= (lo || ragged ? 10 : 7) * cus;
    const bool big = a.max_new >= 512 && 8 * large >= 5 * cus && pays;
    // Two sets of waves (prefill_halves_kernel) while every CU has one workgroup of 128 columns at most; on short contexts the
    // larger start and the sums' exchange cost more than half of a chain, and beyond one a CU a second one waits for the first where it
    // ran beside it.  Graph replay, append included, 128 columns -> this, us (128 columns a CU): ten chunks of 8..372 rows on 345..3355
    // at 16 / 1 heads (1) 84 -> 58, five of 7..495 on 507..6532 at 16 / 2 (0.65) 127 -> 102, five of 141..690 on 385..6190 at 8 / 2 (0.55) 119
    // -> 98, four of 131..302 on 476..2926 (0.97) 44 -> 40, one prompt of 1700 (0.96) 35 -> 32, four at 16 / 1 of up to 664 rows on 500, 30.5
    // -> 28.8, two prompts of 424 on pages of 64 (0.85) 23.9 -> 24.1; but 13 prompts of 57..180 at 16 / 1 (0.8) 14.3 -> 16.1, five of 223..342 at
    // 16 / 2 (0.73) 16.2 -> 17.5, 31 chunks of 26..110 on 765..948 at 16 / 1 (1.04) 38.8 -> 47.4, five of 46..532 on 1187..3571 (1.2) 87 -> 92 (but 26
    // of about 300 on 130..3153 at 4 / 4, pages of 32 (1.35) 137 -> 100), nine prompts of 400 (1.7) 24.0 -> 30.5.
    const bool halves = !big && a.max_ctx >= 512 && a.c.hkv * tiles_bound(a, 128) <= cus;
    if (halves) return !lo ? launch_prefill_halves<128, false, true>(a, st) : a.c.d == 128 ? launch_prefill_halves<128, true, false>(a, st) : launch_prefill_halves<64, true, false>(a, st);
    if (!lo) return big ? launch_prefill_nw<8, 128, false, true>(a, st) : launch_prefill_nw<4, 128, false, true>(a, st);
    if (a.c.d == 128) return big ? launch_prefill_nw<8, 128, true, false>(a, st) : launch_prefill_nw<4, 128, true, false>(a, st);
    return launch_prefill_nw<4, 64, true, false>(a, st);
}

ag_status launch_prefill_mfma(const AttnArgs& a, hipStream_t st) { return launch_tiles(a, false, st); }
ag_status launch_prefill_mfma_lo(const AttnArgs& a, hipStream_t st) { return launch_tiles(a, true, st); }

}  // namespace ag
