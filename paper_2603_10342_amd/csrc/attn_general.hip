// General paged softmax attention in fp32 arithmetic: any supported head_dim,
// page size and storage dtype, for all three request classes (paper Sec. I,
// Sec. II-A): row i of session s sits at position P_s + i and sees keys
// 0 .. P_s + i; a decode step is the one-row case at position ctx_len - 1.
//
// One wavefront per (row, query head).  Keys are taken 64 at a time, one per
// lane (score = scale * q.k in fp32, then a streaming softmax: running max m,
// running sum l, accumulator rescaled when m grows); values are accumulated
// with lane = channel.  It is the path for what the other kernels do not
// cover (pages below 16 tokens, pointers off 16 bytes) and for calls of few keys
// and rows (rows_preferred()); it is not tuned.
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

// Calls of so few keys and rows that starting a workgroup per (session, KV head) pair, which is what the other kernels do, takes
// longer than one wave per (row, head).  Two things have to hold.  Throughput: rows of a pair times (8 + keys), a row's time in
// units of a key's, at most `rows`.  Latency: a wave goes through its keys one after another, so `key` pairs a key after the
// first `pairs` of them (on 256 CUs; others in proportion).  Kernels padded to 64, 128 or 256 channels pay for the padding, fp32 at
// 256 for spilled registers too, and lose to rows earlier: below 0 pairs even with one session.  One fp32 row a pair leaves most of a
// padded tile empty at any context; there latency alone decides.
// Both sides were measured at 1560 decode and 3120 resume batches (1 to 2048 sessions, 1 to 201 keys, 1 to 4 rows, groups of 1, 4 and
// 16, bf16 and fp32 at 8, 64, 128, 136 and 256 channels).  What the lines choose is on average within 0.3 % (bf16 unpadded) to 2.4 %
// (fp32 padded) of the faster side.  The other kernel | this one, us.  Decode, 32 / 8 heads: 64 sessions of 4 tokens, bf16 64 7.1 |
// 7.6, fp32 128 16 | 12; 256 of 16, bf16 64 23 | 22, bf16 128 34 | 38; 64 of 8, fp32 136 36 | 16, bf16 8 8.0 | 6.5; one of one token,
// fp32 136 16 | 9.  Resume of one row, 32 / 32 heads: 16 sessions of 61 tokens, bf16 64 8.7 | 23, bf16 256 19 | 67; 256 of 32, bf16
// 128 115 | 70; 256 of 501, fp32 136 4533 | 2189, fp32 72 1402 | 1097.
namespace {
struct Line { int rows, key, pairs; };
constexpr Line kLines[2][2][2] = {   // [decode][padded][fp32]
    {{{80, 32, 512}, {112, 20, 0}}, {{144, 32, -128}, {208, 16, -128}}},
    {{{64, 24, 512}, {64, 20, 128}}, {{208, 32, -128}, {256, 16, -128}}},
};
}  // namespace

static bool rows_preferred(const AttnArgs& a, hipStream_t st)
{
    const bool padded = a.c.d != 64 && a.c.d != 128 && a.c.d != 256, f32 = a.c.dtype == AG_F32;
    const Line& line = kLines[a.ctx_lens ? 1 : 0][padded ? 1 : 0][f32 ? 1 : 0];
    const int64_t pair_rows = (int64_t)a.total_rows * (a.hq / a.c.hkv);          // rows of all sessions' pairs with one KV head
    const bool one_row = !a.ctx_lens && padded && f32 && pair_rows <= a.batch;
    if (!one_row && pair_rows * (8 + (int64_t)a.max_ctx) > (int64_t)line.rows * a.batch) return false;
    return (int64_t)line.key * a.max_ctx <= (int64_t)a.batch * a.c.hkv * 256 / stream_cus(st) - line.pairs;
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
