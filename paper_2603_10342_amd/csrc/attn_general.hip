// General paged softmax attention in fp32 arithmetic: any supported head_dim,
// page size and storage dtype, for all three request classes (paper Sec. I,
// Sec. II-A): row i of session s sits at position P_s + i and sees keys
// 0 .. P_s + i; a decode step is the one-row case at position ctx_len - 1.
//
// One wavefront per (row, query head).  Keys are taken 64 at a time, one per
// lane (score = scale * q.k in fp32, then a streaming softmax: running max m,
// running sum l, accumulator rescaled when m grows); values are accumulated
// with lane = channel.  It is the path for what the other kernels do not
// cover (pages below 16 tokens, pointers off 16 bytes); it is not tuned.
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

ag_status launch_attn_general(const AttnArgs& a, hipStream_t st)
{
    if (a.ctx_lens && decode_any_supported(a)) return launch_decode_any(a, st);
    if (!a.ctx_lens && prefill_any_supported(a)) return launch_prefill_any(a, st);
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
