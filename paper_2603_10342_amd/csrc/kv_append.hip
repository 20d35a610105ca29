// KV append (paper Sec. II-A: the prefill builds the KV cache; Sec. III-C: the
// cache is one pool shared by the prefill and decode sides) and the placement
// probe used to check CU masks.
//
// Append is an index map plus a bit-exact copy: new token i of session s goes
// to logical position P_s + i -> page bt[s][pos / ps], slot pos % ps.
//   K page  [D/8][slot][8] : chunk-major; a token's row is cut into 8-channel chunks
//   V page  [slot/8'][D][8]: transposed in chunks of 8 keys, see v_offset()
// HBM-bound: 2 * T * 2*Hkv*D*sizeof bytes (read + write).  Two kernels:
//   kv_append_groups_kernel pages of 16 tokens or more: one workgroup per (touched 16-token group, KV head), rows staged in LDS
//   kv_append_kernel        smaller pages, and many sessions of a few rows: one workgroup of 256 threads takes 16
//                           consecutive rows of the token-major input and one KV head; 16 neighbouring lanes hold 16
//                           consecutive tokens of one chunk of D, so each store instruction writes runs of
//                           neighbouring slots.
#include <algorithm>

#include "ag_internal.h"
#include "find_session.h"

namespace ag {

namespace {

constexpr int kTok = 16;   // tokens per workgroup

// E is the raw storage element (uint16_t for bf16, uint32_t for fp32).
template <typename E>
struct alignas(16) Chunk8 { E e[8]; };
typedef uint32_t Words16 __attribute__((ext_vector_type(4)));

template <typename E>
__global__ __launch_bounds__(256) void kv_append_kernel(E* __restrict__ k_pool, E* __restrict__ v_pool,
                                                        const E* __restrict__ k_new, const E* __restrict__ v_new,
                                                        const int32_t* __restrict__ bt, int max_pages,
                                                        const int32_t* __restrict__ prefix_lens,
                                                        const int32_t* __restrict__ new_lens,
                                                        const int32_t* __restrict__ cu_new, int batch, int total_new,
                                                        int hkv, int d, int ps, int ps_shift)
{
    __shared__ int64_t s_page[kTok];   // physical page of each of the 16 tokens, -1 if past the end
    __shared__ int s_slot[kTok];

    const int tid = threadIdx.x;
    const int t0 = blockIdx.x * kTok;
    const int h = blockIdx.y;

    if (tid < kTok) {
        const int t = t0 + tid;
        int64_t page = -1;
        int slot = 0;
        if (t < total_new) {
            // session s with cu_new[s] <= t < cu_new[s+1]; empty sessions are stepped over
            int lo = 0, hi = batch;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (cu_new[mid] <= t) lo = mid; else hi = mid;
            }
            const int s = lo, i = t - cu_new[s];
            const int pos = prefix_lens[s] + i;
            if (i < new_lens[s]) {                  // total_new may be a bound: a row of nobody's past the last session's
                page = bt[(int64_t)s * max_pages + (pos >> ps_shift)];
                slot = pos & (ps - 1);
            }
        }
        s_page[tid] = page;
        s_slot[tid] = slot;
    }
    __syncthreads();

    const int chunks = d >> 3;   // 8-element chunks per row
    using C8 = Chunk8<E>;

    // thread (token = tid % 16, chunk = tid / 16 + 16*r): 16 neighbouring lanes hold 16 consecutive
    // tokens of one chunk, so both stores below write runs of neighbouring slots
    const int tok = tid & 15;
    const int64_t page = s_page[tok];
    if (page >= 0) {
        const int slot = s_slot[tok];
        const int64_t row = (int64_t)(t0 + tok) * hkv + h;
        E* kdst = k_pool + ((int64_t)page * hkv + h) * d * ps + (int64_t)slot * 8;        // + chunk * ps * 8
        E* vdst = v_pool + ((int64_t)page * hkv + h) * d * ps;
        for (int c = tid >> 4; c < chunks; c += 16) {
            *reinterpret_cast<C8*>(kdst + (int64_t)c * ps * 8) = *reinterpret_cast<const C8*>(k_new + row * d + c * 8);
            const C8 x = *reinterpret_cast<const C8*>(v_new + row * d + c * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) vdst[v_offset(slot, c * 8 + e, ps, d)] = x.e[e];
        }
    }
}

// Group-wise append for pages of 16 tokens or more.  One workgroup per (touched 16-token group of a session, KV head):
// the group's new tokens are read row by row (coalesced) into LDS and written out in the pool layouts with
// 16/32-byte stores: K as runs of neighbouring slots per chunk, V - when the whole group is new, the usual case
// in a prefill - as whole 8-key chunks, 2 KiB contiguous per wave.  A partly filled group (the first and last
// of an appended range, or a decode step's single token) writes V element by element so that slots that
// already hold older tokens are not touched.
// Items are numbered session-major; every wave finds the workgroup's session itself (find_session()), its lengths fetched
// along: the rows, and the page id, are requested one memory round trip after the kernel starts for up to 64 sessions, which
// is what bounds an append of few tokens.
template <typename E>
__global__ __launch_bounds__(256) void kv_append_groups_kernel(E* __restrict__ k_pool, E* __restrict__ v_pool,
                                                               const E* __restrict__ k_new, const E* __restrict__ v_new,
                                                               const int32_t* __restrict__ bt, int max_pages,
                                                               const int32_t* __restrict__ prefix_lens,
                                                               const int32_t* __restrict__ new_lens,
                                                               const int32_t* __restrict__ cu_new, int batch, int hkv,
                                                               int d, int ps, int ps_shift)
{
    constexpr int kGroup = 16;
    using C8 = Chunk8<E>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    C8* lds_k = reinterpret_cast<C8*>(smem);                       // [16 tokens][d/8]
    C8* lds_v = lds_k + kGroup * (d >> 3);

    const int tid = threadIdx.x, item = blockIdx.x, h = blockIdx.y;
    const int chunks = d >> 3;

    // a session has at most as many groups as tokens, and at most N / 16 + 2: both summed over the sessions before
    const Session f = find_session(new_lens, prefix_lens, cu_new, batch, item, [](int ss, int cu) { return min(cu, (cu >> 4) + 2 * ss); });
    const int s = f.s, last_pos = f.prefix + f.new_len - 1, grp = (f.prefix >> 4) + (item - f.first);
    if (f.new_len <= 0 || grp > last_pos >> 4) return;               // nobody's item
    const int pos0 = max(f.prefix, grp << 4), n_tok = min(last_pos, (grp << 4) + 15) - pos0 + 1;     // uniform
    const int row0 = f.row0 + (pos0 - f.prefix);
    const int64_t page = bt[(int64_t)s * max_pages + (pos0 >> ps_shift)];
    const int slot0 = pos0 & (ps - 1);                               // in the page

    auto page_of = [&](E* pool) { return pool + (page * hkv + h) * (int64_t)d * ps; };
    if (n_tok > 1) {
        for (int idx = tid; idx < n_tok * chunks; idx += 256) {          // rows in, 16 lanes per 8-chunk run
            const int row = idx / chunks, c = idx - row * chunks;
            const int64_t src = ((int64_t)(row0 + row) * hkv + h) * d + c * 8;
            lds_k[idx] = *reinterpret_cast<const C8*>(k_new + src);
            lds_v[idx] = *reinterpret_cast<const C8*>(v_new + src);
        }
        __syncthreads();

        E *kpage = page_of(k_pool), *vpage = page_of(v_pool);
        for (int idx = tid; idx < n_tok * chunks; idx += 256) {          // K: neighbouring lanes, neighbouring slots
            const int c = idx / n_tok, i = idx - c * n_tok;
            *reinterpret_cast<C8*>(kpage + ((int64_t)c * ps + slot0 + i) * 8) = lds_k[i * chunks + c];
        }
        const E* lv = reinterpret_cast<const E*>(lds_v);                 // [token][d]
        if (n_tok == kGroup) {                                           // whole group: V as 8-key chunks
            for (int idx = tid; idx < 2 * d; idx += 256) {
                const int half = idx / d, ch = idx - half * d;
                C8 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x.e[e] = lv[(half * 4 + e) * d + ch];
                    x.e[4 + e] = lv[(8 + half * 4 + e) * d + ch];
                }
                *reinterpret_cast<C8*>(vpage + ((int64_t)((slot0 >> 3) + half) * d + ch) * 8) = x;
            }
        } else {
            for (int idx = tid; idx < n_tok * d; idx += 256) {
                const int ch = idx / n_tok, i = idx - ch * n_tok;
                vpage[v_offset(slot0 + i, ch, ps, d)] = lv[i * d + ch];
            }
        }
        return;
    }
    // A decode's token: straight through registers.  What such an append costs is its stores, a few bytes in each of many lines.
    // Marked non-temporal they need no write-back at the end of the kernel, but the attention that follows reads these lines from
    // further away, which a step of few workgroups waits for.  Append and decode, graph replay, through LDS / registers / registers
    // and marked, bf16 on 8 KV heads: 32 sessions of 100 to 800 tokens, 256 channels 31.6, 31.3, 29.9 us, 128 15.7, 15.4, 14.8; 64 of
    // 1023 to 4095 118.9, 118.8, 117.3; 8 of 300 to 900 (64 workgroups), 256 channels 21.7, 21.5, 21.2; 2 of 91 to 365 12.7, 12.5,
    // 12.7, 128 6.8, 6.6, 6.9.  (Longer runs gain nothing from the mark: 211 rows on 6007 tokens 36.2 -> 36.6.)
    auto one_token = [&](auto put) {
        E *kpage = page_of(k_pool), *vpage = page_of(v_pool);
        const int64_t src = ((int64_t)row0 * hkv + h) * d;
        C8 k;
        E v = 0;
        if (tid < chunks) k = *reinterpret_cast<const C8*>(k_new + src + tid * 8);
        if (tid < d) v = v_new[src + tid];
        if (tid < chunks) {
            Words16* dst = reinterpret_cast<Words16*>(kpage + ((int64_t)tid * ps + slot0) * 8);
#pragma unroll
            for (int i = 0; i < (int)(sizeof(C8) / 16); ++i) put(reinterpret_cast<const Words16*>(&k)[i], dst + i);
        }
        if (tid < d) put(v, vpage + v_offset(slot0, tid, ps, d));
    };
    if (gridDim.x * gridDim.y < 64) {
        one_token([](auto x, auto* dst) { *dst = x; });
    } else {
        asm volatile("");                // (keeps the compiler from making one of the two)
        one_token([](auto x, auto* dst) { __builtin_nontemporal_store(x, dst); });
        asm volatile("");
    }
}

// Where did this workgroup run?  HW_ID (register 4): CU id bits 8-11, shader
// array bit 12, shader engine bits 13-15; XCC_ID (register 20): bits 0-3.
__global__ __launch_bounds__(64) void probe_kernel(uint32_t* ids, int spin_cycles)
{
    const long long t_end = (long long)clock64() + spin_cycles;
    int guard = 0;
    while ((long long)clock64() < t_end && guard < (1 << 24)) ++guard;   // bounded: always terminates
    if (threadIdx.x == 0) {
        const uint32_t hw = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 4);
        const uint32_t xcc = __builtin_amdgcn_s_getreg((31 << 11) | (0 << 6) | 20);
        const uint32_t cu = (hw >> 8) & 0xF, sa = (hw >> 12) & 0x1, se = (hw >> 13) & 0x7;
        ids[blockIdx.x] = cu | (sa << 8) | (se << 12) | ((xcc & 0xF) << 16);
    }
}

}  // namespace

ag_status launch_kv_append(const CacheView& c, const void* k_new, const void* v_new, const int32_t* bt, int max_pages,
                           const int32_t* prefix_lens, const int32_t* new_lens, const int32_t* cu_new, int batch,
                           int total_new, hipStream_t st)
{
    // every session touches at most N_s / 16 + 2 groups, and every group has a token
    const int64_t items = std::min<int64_t>(total_new / 16 + 2 * (int64_t)batch, total_new);
    if (c.ps >= 16 && (items > 0x7fffffff || c.hkv > 65535)) { set_error("append too large for one launch"); return AG_ERR_INVALID_ARG; }
    const size_t row_bytes = (size_t)c.d * (c.dtype == AG_BF16 ? 2 : 4);
    // More groups than the chip holds at once (256 CUs of eight workgroups), each mostly empty: a workgroup that takes 16 rows of
    // whatever sessions comes to fewer.  It is the slower one per byte: rows up to 256 bytes, 2 KiB of them a session.  Sessions
    // x rows each, 8 KV heads, us by groups -> by rows.  128 bytes a row: 100x4 (1800 groups) 4.6 -> 4.9, 300x4 (5400) 7.9 ->
    // 6.5, 300x15 12.0 -> 12.2, 2048x4 37 -> 22.  256: 300x1 6.4 -> 7.1, 300x2 9.5 -> 8.0, 300x8 12.1 -> 11.9, 300x15 16.1 -> 17.7,
    // 1000x4 23.7 -> 19.5.  512: 300x2 11.4 -> 12.3, 300x4 12.2 -> 14.9, 1000x1 16.1 -> 19.6.
    const bool by_rows = items * c.hkv > 2048 && row_bytes <= 256 && (int64_t)total_new * (int64_t)row_bytes <= 2048 * (int64_t)batch;
    if (c.ps >= 16 && !by_rows) {
        const dim3 grid((unsigned)items, c.hkv);
        const size_t lds = 2 * 16 * row_bytes;
        if (c.dtype == AG_BF16)
            hipLaunchKernelGGL(kv_append_groups_kernel<uint16_t>, grid, dim3(256), lds, st, (uint16_t*)c.k, (uint16_t*)c.v,
                               (const uint16_t*)k_new, (const uint16_t*)v_new, bt, max_pages, prefix_lens, new_lens,
                               cu_new, batch, c.hkv, c.d, c.ps, c.ps_shift);
        else
            hipLaunchKernelGGL(kv_append_groups_kernel<uint32_t>, grid, dim3(256), lds, st, (uint32_t*)c.k, (uint32_t*)c.v,
                               (const uint32_t*)k_new, (const uint32_t*)v_new, bt, max_pages, prefix_lens, new_lens,
                               cu_new, batch, c.hkv, c.d, c.ps, c.ps_shift);
        return hip_check(hipGetLastError(), "kv_append launch");
    }
    const dim3 grid((total_new + kTok - 1) / kTok, c.hkv);
    if (c.dtype == AG_BF16) {
        hipLaunchKernelGGL(kv_append_kernel<uint16_t>, grid, dim3(256), 0, st, (uint16_t*)c.k, (uint16_t*)c.v,
                           (const uint16_t*)k_new, (const uint16_t*)v_new, bt, max_pages, prefix_lens, new_lens, cu_new, batch,
                           total_new, c.hkv, c.d, c.ps, c.ps_shift);
    } else {
        hipLaunchKernelGGL(kv_append_kernel<uint32_t>, grid, dim3(256), 0, st, (uint32_t*)c.k, (uint32_t*)c.v,
                           (const uint32_t*)k_new, (const uint32_t*)v_new, bt, max_pages, prefix_lens, new_lens, cu_new, batch,
                           total_new, c.hkv, c.d, c.ps, c.ps_shift);
    }
    return hip_check(hipGetLastError(), "kv_append launch");
}

ag_status launch_probe(uint32_t* ids_out, int n_wg, int spin_cycles, hipStream_t st)
{
    hipLaunchKernelGGL(probe_kernel, dim3(n_wg), dim3(64), 0, st, ids_out, spin_cycles);
    return hip_check(hipGetLastError(), "probe launch");
}

}  // namespace ag
