"""bf16 / 128 / page 16 decode in shares: what a step's arithmetic and the cuts of the shares promise, read from the workspace that
the split kernel leaves behind, and both forms of the step against the fp64 oracle in shares of up to 128 steps."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, i32, make_cache, to_dev, to_f64
from helpers import fresh_pools, make_batch, oracle_append
from oracle import oracle as O
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I
from test_gpu_decode_step import both_ways, same_bits, step_workspace

pytestmark = pytest.mark.gpu

STEP, MIN_STEPS, MAX_STEPS = 32, 8, 128


def split_workspace(batch, g, max_ctx):
    """The workspace of ag_attn_decode, and where its parts lie: [share, steps before each session], O, (m, l)."""
    ws = torch.zeros(B.ag_attn_decode_workspace_bytes(batch, g.num_q_heads, g.head_dim, max_ctx) // 4, dtype=torch.float32, device="cuda")
    pieces = ((max_ctx + STEP - 1) // STEP - 1) // MIN_STEPS + 2
    header = (batch + 4) & ~3
    ml = header + batch * g.num_q_heads * pieces * g.head_dim
    return ws, pieces, ml


def test_equal_scores_have_equal_weights():
    """Every key the same and a score that rounding changes: each weight is exactly 1, and a part's sum the number of its tokens."""
    g = I.Geometry(16, 1, 128, 16, 100, I.BF16)
    ctx = 1300
    fill = make_batch(g, [0], [ctx], seed=81, sigma_qk=2.5, sigma_v=1.0)
    fill.k_new[:] = fill.k_new[:1]
    cache = make_cache(g)
    df = DevBatch(fill)
    gpu_append(cache, df)
    q = df.q[:1].contiguous()
    ws, pieces, ml = split_workspace(1, g, ctx)
    B.ag_attn_decode(cache, q, torch.empty_like(q), df.bt, i32([ctx]), ctx, g.num_q_heads, g.scale, ws)
    torch.cuda.synchronize()
    share = int(ws[:1].view(torch.int32)[0])
    m, l = ws[ml:ml + 16 * pieces * 2].view(16, pieces, 2).cpu().numpy().transpose(2, 0, 1)
    used = -(-ctx // (share * STEP))
    assert share == MIN_STEPS and np.abs(m[:, 0]).max() > 16           # half a unit in the last place there is 1e-6, ten times that of a weight
    assert np.array_equal(l[:, :used], np.broadcast_to(np.minimum(share * STEP, ctx - np.arange(used) * share * STEP), (16, used)).astype(np.float32))


@pytest.mark.parametrize("lo,hi,bound", [(3000, 6000, 6000), (200, 400, 6000), (40, 4500, 16000)])
def test_shares_of_at_most_128_steps_on_eight_cus(lo, hi, bound):
    """Twelve sessions on eight CUs, more shares than two a CU; then contexts far below the bound."""
    g = I.Geometry(8, 2, 128, 16, 6000, I.BF16)
    c = I.make_decode(batch=12, lo=lo, hi=hi, num_pages=g.num_pages, geom=g, seed=82, sigma_qk=1.0, sigma_v=1.0)
    bound = max(bound, int(c.ctx_lens.max()))
    kp, vp = fresh_pools(g)
    for b in (c.fill, c.step):
        oracle_append(kp, vp, b)
    ref = O.decode(kp, vp, g.dtype, c.step.q, c.block_tables, c.ctx_lens, g.num_q_heads, g.scale)
    stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, 1))
    try:
        c1, out1, c2, out2, _, _ = both_ways(g, c.fill, c.step, stream=stream)
        check_close(to_f64(out1, g.dtype), ref, g.dtype, "step")
        assert same_bits(out1, out2) and same_bits(c1.k_pool, c2.k_pool) and same_bits(c1.v_pool, c2.v_pool)
        table = np.zeros((12, max(-(-bound // 16), c.block_tables.shape[1])), np.int32)
        table[:, :c.block_tables.shape[1]] = c.block_tables
        ws, _, _ = split_workspace(12, g, bound)
        q, out = to_dev(c.step.q, g.dtype), torch.empty_like(out1)
        torch.cuda.synchronize()
        B.ag_attn_decode(c2, q, out, i32(table), i32(c.ctx_lens), bound, g.num_q_heads, g.scale, ws, stream=stream)
        torch.cuda.synchronize()
        check_close(to_f64(out, g.dtype), ref, g.dtype, "decode")
        share = int(ws[:1].view(torch.int32)[0])
    finally:
        torch.cuda.synchronize()
        B.ag_stream_destroy(stream)
    steps = 2 * int(sum(-(-int(x) // STEP) for x in c.ctx_lens))
    most = 2 * 12 * -(-bound // STEP)
    shares = 16 * -(-most // (16 * MAX_STEPS))                         # two workgroups a CU, as many rounds of them as 128 steps ask for
    assert share == max(MIN_STEPS, -(-steps // shares)) <= MAX_STEPS


@pytest.mark.parametrize("step", [True, False])
@pytest.mark.parametrize("ctx", [100, 256, 500, 512])
def test_one_workgroup_a_pair_rounds_no_step_s_largest_weight(ctx, step):
    """One key of every 32 counts, the odd steps' at exp(-0.2): a weight against its step's own maximum is 1 and exact.  Values of 1
    and of about -exp(0.2) leave a result near the rounding of such a weight to bf16, 2^-9, so that one that is rounded shows."""
    g = I.Geometry(16, 1, 128, 16, 40, I.BF16)
    low, value = I.stored_to_f64(I.store(np.array([-0.2, -1.22], np.float32), I.BF16), I.BF16)
    fill = make_batch(g, [0], [ctx], seed=83, sigma_qk=1.0, sigma_v=1.0)
    k, v, q = np.zeros((ctx, 1, 128), np.float32), np.ones((ctx, 1, 128), np.float32), np.zeros((ctx, 16, 128), np.float32)
    k[:, 0, 0] = -200
    k[7::64, 0, 0] = 0
    k[39::64, 0, 0] = low
    v[32:] = np.where(np.arange(32, ctx) // 32 % 2 == 1, value, 1)[:, None, None]
    q[:, :, 0] = 1
    fill = make_batch(g, [0], [ctx], seed=83, k=k, v=v, q=q)
    even, odd = len(range(7, ctx, 64)), len(range(39, ctx, 64))
    want = (even + odd * value * np.exp(low)) / (even + odd * np.exp(low))
    df = DevBatch(fill)
    cache = make_cache(g)
    qn = df.q[-1:].contiguous()
    out = torch.empty_like(qn)
    gpu_append(cache, df)
    if step:
        ws, _ = step_workspace(1, g, ctx)
        B.ag_decode_step(cache, df.k_new[-1:].contiguous(), df.v_new[-1:].contiguous(), qn, out, df.bt, i32([ctx]), ctx, 16, 1.0, ws)
    else:
        B.ag_attn_decode(cache, qn, out, df.bt, i32([ctx]), ctx, 16, 1.0, split_workspace(1, g, ctx)[0])
    torch.cuda.synchronize()
    got = to_f64(out, g.dtype)
    # the result's own rounding, and sums in fp32 of up to 16 numbers of 1 that cancel to it
    assert np.all(np.abs(got - want) <= 2.0 ** -9 * abs(want) + 16 * 2.0 ** -24 * 1.22), (got.reshape(-1)[:4], want)
