"""Batches of many short sessions: every item finds its session, and no call takes longer than one wave per (row, head) would."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_decode, gpu_prefill, gpu_resume, make_cache, pools_match
from helpers import fresh_pools, make_batch, oracle_append, oracle_attn
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


def graph_time(call, calls=20):
    """Shortest replay of a graph of `calls` calls."""
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(calls):
                call()
        best = 1e9
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record(stream)
            graph.replay()
            end.record(stream)
            end.synchronize()
            best = min(best, start.elapsed_time(end))
    return best / calls


def off_16_bytes(q):
    """The same q at an address that only one wave per (row, head) takes."""
    off = torch.empty(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view(q.shape)
    off.copy_(q)
    return off


def table_pages(ctx, ps):
    return int(sum((max(int(c), 1) + ps - 1) // ps for c in ctx)) + 3


# 8 KV heads: groups of 16 tokens against 16 rows of whatever sessions.  (rows a session, sessions) on both sides of 2048 groups
# (3 rows: 86 sessions) and of 2 KiB of keys a session (bf16 64: 16 rows, bf16 128 and fp32 64: 8); 257, 2100 and 4100 sessions
# are looked up in two and three steps
@pytest.mark.parametrize("dtype,d,ps,hkv", [(I.BF16, 64, 32, 8), (I.BF16, 128, 16, 8), (I.F32, 64, 64, 8), (I.F32, 128, 16, 8), (I.BF16, 24, 16, 1)])
@pytest.mark.parametrize("batch,rows", [(85, 3), (86, 3), (257, 1), (257, 4), (200, 8), (200, 9), (200, 16), (200, 17), (2100, 2), (4100, 1)])
def test_append_of_many_sessions_bit_exact(batch, rows, dtype, d, ps, hkv):
    """Ragged chunks, empty ones among them; total_new as it is and as a bound that is 50 too large (lengths that change under a
    captured graph).  Slots outside of the chunks stay NaN."""
    rng = np.random.default_rng(73 + batch)
    p, n = rng.integers(0, 40, size=batch).astype(np.int32), rng.integers(0, 2 * rows + 1, size=batch).astype(np.int32)
    n[[0, batch - 1]] = [0, rows]
    ctx = p + n
    g = I.Geometry(hkv, hkv, d, ps, table_pages(ctx, ps), dtype)
    b = make_batch(g, p, n, seed=73, bt=I.deal_block_tables(I.rng_for(73, 0), np.maximum(ctx, 1), ps, g.num_pages))
    kp, vp = fresh_pools(g)
    oracle_append(kp, vp, b)
    dev = DevBatch(b)
    for total in (dev.total, dev.total + 50):
        cache = make_cache(g)
        B.ag_kv_append(cache, dev.k_new, dev.v_new, dev.bt, dev.prefix, dev.new, dev.cu, total)
        pools_match(cache, kp, vp, dtype)


@pytest.mark.parametrize("d,ps", [(64, 32), (128, 16)])
def test_append_to_a_thousand_sessions_costs_little_more_than_to_a_hundred(d, ps):
    """2000 rows (1.3 and 1.6 times measured; 8.7 and 7.3 where every workgroup added the lengths up)."""
    times = []
    for batch in (1000, 100):
        p, n = np.full(batch, 20, np.int32), np.full(batch, 2000 // batch, np.int32)
        g = I.Geometry(8, 8, d, ps, table_pages(p + n, ps), I.BF16)
        cache, b = make_cache(g, poison=False), DevBatch(make_batch(g, p, n, seed=76, bt=I.deal_block_tables(I.rng_for(76, 0), p + n, ps, g.num_pages)))
        times.append(graph_time(lambda: B.ag_kv_append(cache, b.k_new, b.v_new, b.bt, b.prefix, b.new, b.cu, b.total)))
    assert times[0] <= 3 * times[1], times


# 64 sessions are looked up in one step, 65 to 4096 in two, more in three
@pytest.mark.parametrize("batch", [64, 65, 256, 257, 1025, 2100, 4100])
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [(I.BF16, 128, 16, 8, 2), (I.BF16, 64, 32, 4, 4), (I.BF16, 128, 32, 2, 1), (I.BF16, 72, 16, 3, 1),
                                               (I.F32, 64, 16, 2, 2), (I.F32, 128, 16, 1, 1), (I.F32, 24, 16, 2, 1)])
def test_every_session_gets_its_rows(batch, dtype, d, ps, hq, hkv):
    """Empty chunks among them, a whole step's share of 64 and the ends of the batch; long chunks in the middle, at the front
    and at the back (tiles of one session over several workgroups)."""
    rng = np.random.default_rng(71 + batch)
    n = rng.integers(0, 5, size=batch).astype(np.int32)
    n[rng.integers(0, batch, size=batch // 3)] = 0
    n[64:128] = 0
    n[[0, 1, batch // 2, batch - 2, batch - 1]] = [140, 1, 33, 70, 2]
    p = rng.integers(0, 20, size=batch).astype(np.int32)
    g = I.Geometry(hq, hkv, d, ps, table_pages(p + n, ps), dtype)
    bt = I.deal_block_tables(I.rng_for(71, 0), np.maximum(p + n, 1), ps, g.num_pages)
    fill, chunk = make_batch(g, np.zeros_like(p), p, seed=71, bt=bt), make_batch(g, p, n, seed=71, bt=bt, stream=2)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    df, db = DevBatch(fill), DevBatch(chunk)
    gpu_append(cache, df)
    oracle_append(kp, vp, fill)
    check_close(gpu_prefill(cache, df), oracle_attn(kp, vp, fill), dtype, f"cold, {batch} sessions")
    gpu_append(cache, db)
    oracle_append(kp, vp, chunk)
    check_close(gpu_resume(cache, db), oracle_attn(kp, vp, chunk), dtype, f"resume, {batch} sessions")


def resume_times(batch, g, p, n):
    p, n = np.full(batch, p, np.int32), np.full(batch, n, np.int32)
    bt = I.deal_block_tables(I.rng_for(72, 0), p + n, g.page_size, g.num_pages)
    cache, b = make_cache(g, poison=False), DevBatch(make_batch(g, p, n, seed=72, bt=bt))
    gpu_append(cache, b)
    return [graph_time(lambda: B.ag_attn_resume(cache, q, b.out, b.bt, b.prefix, b.new, b.cu, b.total, b.max_new, b.max_ctx, g.num_q_heads,
                                                g.scale)) for q in (b.q, off_16_bytes(b.q))]


def test_the_lookup_of_thousands_of_sessions_costs_less_than_their_rows():
    """2048 sessions of one row on three tokens, 16 query heads on one KV head: against the same call with one wave per (row,
    head) (0.5 of its time measured; 1.4 where every workgroup added the lengths up, 256 sessions at a time)."""
    tiles, row_by_row = resume_times(2048, I.Geometry(16, 1, 64, 16, 2051, I.BF16), 3, 1)
    assert tiles <= 0.9 * row_by_row


# 1200 pairs of one row.  Keys on both sides of the lines between one wave per (row, head) and the other kernels: resume bf16 21,
# fp32 60, padded bf16 41, padded fp32 83; decode bf16 28, fp32 53, padded as resume, and 256 tokens a CU 54
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [(I.BF16, 64, 32, 4, 4), (I.BF16, 128, 32, 4, 4), (I.BF16, 256, 16, 4, 4), (I.BF16, 72, 32, 4, 4),
                                               (I.F32, 128, 16, 4, 4), (I.F32, 72, 64, 4, 4)])
@pytest.mark.parametrize("ctx", [3, 21, 22, 28, 29, 41, 42, 53, 54, 55, 60, 61, 83, 84])
def test_crowds_at_the_line_to_row_by_row(ctx, dtype, d, ps, hq, hkv):
    """300 sessions of one row, one of them of one token, one empty."""
    c = np.full(300, ctx, np.int32)
    c[[0, 7, 299]] = [1, ctx // 2, 0]
    g = I.Geometry(hq, hkv, d, ps, table_pages(c, ps), dtype)
    bt = I.deal_block_tables(I.rng_for(74, 0), np.maximum(c, 1), ps, g.num_pages)
    n = np.minimum(c, 1).astype(np.int32)
    fill, last = make_batch(g, np.zeros_like(c), c - n, seed=74, bt=bt), make_batch(g, c - n, n, seed=74, bt=bt, stream=2)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    df, dl = DevBatch(fill), DevBatch(last)
    gpu_append(cache, df)
    oracle_append(kp, vp, fill)
    gpu_append(cache, dl)
    oracle_append(kp, vp, last)
    ref = oracle_attn(kp, vp, last)
    check_close(gpu_resume(cache, dl), ref, dtype, f"resume of one row on {ctx}")
    q = torch.zeros((300, hq, d), dtype=dl.q.dtype, device="cuda")
    q[torch.from_numpy(np.nonzero(c > 0)[0]).cuda()] = dl.q
    got = gpu_decode(cache, q, dl.bt, dl.ctx, ctx, g)
    assert np.all(got[c == 0] == 0)
    check_close(got[c > 0], ref, dtype, f"decode of {ctx}")


# 2048 sessions on three tokens: by tiles 1.7 of the time, and 3.4 where every workgroup added the lengths up.  One session of one
# token, fp32 padded to 256 channels: 1.5; 128 of 32 with a KV head for each query head: 2.9.  The last two are for the tiles: one
# wave would go through its keys alone (3 times as long)
@pytest.mark.parametrize("batch,dtype,d,hq,hkv,prefix,share", [(2048, I.BF16, 64, 32, 8, 3, 1.3), (1, I.F32, 136, 32, 8, 1, 1.2),
                                                               (128, I.F32, 136, 32, 32, 32, 1.2), (16, I.BF16, 64, 32, 32, 60, 0.7),
                                                               (128, I.BF16, 128, 4, 4, 60, 0.7)])
def test_one_row_on_a_few_tokens_against_row_by_row(batch, dtype, d, hq, hkv, prefix, share):
    now, row_by_row = resume_times(batch, I.Geometry(hq, hkv, d, 32, 3 + batch * ((prefix + 32) // 32), dtype), prefix, 1)
    assert now <= share * row_by_row


# 64 sessions, the start of as many conversations: by shares of 256 tokens 2.7 of the time at four tokens and 1.3 at 31; fp32 padded
# to 256 channels 1.9 at 11 tokens, one session of one token 1.8
@pytest.mark.parametrize("batch,ctx,dtype,d", [(64, 4, I.BF16, 64), (64, 31, I.BF16, 64), (64, 4, I.F32, 128), (64, 11, I.F32, 136), (1, 1, I.F32, 136)])
def test_decode_of_short_sessions_is_no_slower_than_row_by_row(batch, ctx, dtype, d):
    c = np.full(batch, ctx, np.int32)
    g = I.Geometry(32, 8, d, 32, table_pages(c, 32), dtype)
    bt = I.deal_block_tables(I.rng_for(75, 0), c, 32, g.num_pages)
    cache, b = make_cache(g), DevBatch(make_batch(g, np.zeros_like(c), c, seed=75, bt=bt))
    gpu_append(cache, b)
    ws = torch.empty(B.ag_attn_decode_workspace_bytes(batch, 32, d, ctx) // 4, dtype=torch.float32, device="cuda")
    q = b.q[ctx - 1::ctx].contiguous()
    out = torch.empty_like(q)
    now, row_by_row = [graph_time(lambda: B.ag_attn_decode(cache, x, out, b.bt, b.ctx, ctx, 32, g.scale, ws)) for x in (q, off_16_bytes(q))]
    assert now <= 1.2 * row_by_row
