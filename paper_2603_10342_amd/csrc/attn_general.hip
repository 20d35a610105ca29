// General paged softmax attention in fp32 arithmetic: any supported head_dim,
// page size and storage dtype, for all three request classes (paper Sec. I,
// Sec. II-A): row i of session s sits at position P_s + i and sees keys
// 0 .. P_s + i; a decode step is the one-row case at position ctx_len - 1.
//
// One wavefront per (row, query head).  Keys are taken 64 at a time, one per
// lane (score = scale * q.k in fp32, then a streaming softmax: running max m,
// running sum l, accumulator rescaled when m grows); values are accumulated
// with lane = channel.  It is the path for what the other kernels do not
// cover (pages below 16 tokens, pointers off 16 bytes) and for crowds of sessions
// of a few tokens; it is not tuned.
#include "ag_internal.h"
#include "attn_general_row.h"

namespace ag {

namespace {

template <typename T>
__global__ __launch_bounds__(256) void attn_general_kernel(AttnArgs a)
{
    __shared__ float s_q[4][256];
    const int w = threadIdx.x >> 6;
    const int64_t item = (int64_t)blockIdx.x * 4 + w;
    if (item >= (int64_t)a.total_rows * a.hq) return;   // whole wave leaves; no block barrier is used below
    const int t = (int)(item / a.hq), h = (int)(item % a.hq);
    int s, pos;
    if (a.cu_new == nullptr) {           // decode: one row per session
        s = t;
        pos = a.ctx_lens[s] - 1;
    } else {
        int lo = 0, hi = a.batch;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.cu_new[mid] <= t) lo = mid; else hi = mid;
        }
        s = lo;
        pos = (a.prefix_lens ? a.prefix_lens[s] : 0) + (t - a.cu_new[s]);
    }
    general::attend_row<T>(a, t, h, s, pos, s_q[w]);
}

}  // namespace

// More (session, KV head) pairs than CUs, each with so few keys and rows that a workgroup's start is most of what a pair costs
// the other kernels (11 to 37 ns a pair on a full chip, by dtype and head_dim), while one wave per (row, head) takes 1 to 4 ns
// and 0.1 to 0.4 a key: rows of a pair times (8 + keys) is the row's time in units of a key's.  Measured, 2048 sessions, the
// other kernel -> this one, us.  Chunks: bf16 64, 4 / 4 heads, 3 rows on 8 tokens (57) 92 -> 57, 4 on 28 (160) 90 -> 140;
// 32 / 8 heads, 1 on 3 (48), bf16 64 181 -> 107, bf16 128 234 -> 169, bf16 256 567 -> 306, fp32 128 614 -> 191; 3 on 8 (228) 182 -> 368,
// 240 -> 710, 580 -> 1354, 636 -> 1026; fp32 64, 4 / 2 heads, 3 on 8 (114) 58 -> 75.  Decode: 32 / 8 heads, 4 tokens (48),
// bf16 64 112 -> 87, bf16 128 155 -> 148, fp32 128 253 -> 184; 11 tokens (76) 112 -> 126, 154 -> 248, 252 -> 365; 64 sessions of 4
// tokens 21 -> 8, 26 -> 12, 47 -> 12.
static bool rows_preferred(const AttnArgs& a, hipStream_t st)
{
    const int64_t pair_rows = (int64_t)a.total_rows * (a.hq / a.c.hkv);          // rows of all sessions' pairs with one KV head
    return pair_rows * (8 + (int64_t)a.max_ctx) <= (int64_t)(a.ctx_lens ? 48 : 80) * a.batch && (int64_t)a.batch * a.c.hkv > stream_cus(st);
}

ag_status launch_attn_general(const AttnArgs& a, hipStream_t st)
{
    if (!rows_preferred(a, st)) {
        if (a.ctx_lens && decode_any_supported(a)) return launch_decode_any(a, st);
        if (!a.ctx_lens && prefill_any_supported(a)) return launch_prefill_any(a, st);
    }
    const int64_t items = (int64_t)a.total_rows * a.hq;
    const int64_t blocks = (items + 3) / 4;
    if (blocks > 0x7fffffff) { set_error("too many rows for one launch"); return AG_ERR_INVALID_ARG; }
    prof_before(st);
    if (a.c.dtype == AG_BF16)
        hipLaunchKernelGGL(attn_general_kernel<__bf16>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(attn_general_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, a);
    prof_after(st);
    return hip_check(hipGetLastError(), "attn_general launch");
}

}  // namespace ag
