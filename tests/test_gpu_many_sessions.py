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
