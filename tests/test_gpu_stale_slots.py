"""Slots that no row may see - behind a session's last token, or of later rows of the same chunk - may hold anything, keys
that are not finite included, and cost a row neither its result nor its place in the tiles: the outputs are the same bits
whatever is there (a row that falls back on plain arithmetic has other bits)."""
import pytest
import torch

from gpu_helpers import DevBatch, gpu_decode, gpu_merged, make_cache
from helpers import make_batch
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I
from test_gpu_precision import cus

pytestmark = pytest.mark.gpu

SHAPES = [(I.F32, 64, 16, 8, 2), (I.F32, 128, 16, 6, 2), (I.F32, 128, 32, 4, 4), (I.BF16, 64, 64, 8, 2), (I.BF16, 128, 16, 8, 2),
          (I.BF16, 128, 32, 6, 2), (I.BF16, 256, 16, 4, 2), (I.F32, 72, 16, 4, 2)]


def outputs(g, prefix, new, stale, last_key=None, seed=83):
    """Bits of a resume prefill whose pools held `stale` before; last_key replaces the key of every session's last token."""
    bt = I.deal_block_tables(I.rng_for(seed, 0), [p + n for p, n in zip(prefix, new)], g.page_size, g.num_pages)
    cache = make_cache(g)
    cache.k_pool.fill_(stale)
    cache.v_pool.fill_(stale)
    fill = DevBatch(make_batch(g, [0] * len(prefix), prefix, seed=seed, bt=bt))
    chunk = DevBatch(make_batch(g, prefix, new, seed=seed, bt=bt, stream=2))
    if last_key is not None:
        chunk.k_new[(chunk.cu[1:] - 1).long()] = last_key
    for b in (fill, chunk):
        B.ag_kv_append(cache, b.k_new, b.v_new, b.bt, b.prefix, b.new, b.cu, b.total)
    B.ag_attn_resume(cache, chunk.q, chunk.out, chunk.bt, chunk.prefix, chunk.new, chunk.cu, chunk.total, chunk.max_new, chunk.max_ctx,
                     g.num_q_heads, g.scale)
    torch.cuda.synchronize()
    return chunk.out.clone().view(torch.int32 if g.dtype == I.F32 else torch.int16), chunk


@pytest.mark.parametrize("per_xcd", [0, 1])
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", SHAPES)
def test_what_no_row_may_see_leaves_every_bit(dtype, d, ps, hq, hkv, per_xcd):
    """On the whole device, and on 8 CUs, where the same batch takes the kernels of whole tiles.  Lengths that end inside
    and at the end of a tile of 32 keys and of a 16-token group."""
    g = I.Geometry(hq, hkv, d, ps, 1024 // ps + 64, dtype)
    prefix, new = [0, 33, 100, 31, 0], [150, 130, 61, 1, 64]
    with cus(per_xcd):
        want, chunk = outputs(g, prefix, new, 0.0)
        for stale in (float("nan"), float("inf"), -float("inf")):
            assert torch.equal(outputs(g, prefix, new, stale)[0], want), f"stale slots of {stale}"
        rows = torch.ones(chunk.total, dtype=torch.bool, device="cuda")
        rows[(chunk.cu[1:] - 1).long()] = False                    # the only rows that see the last key
        for key in (float("nan"), float("inf")):
            assert torch.equal(outputs(g, prefix, new, 0.0, last_key=key)[0][rows], want[rows]), f"a later key of {key}"


@pytest.mark.parametrize("per_xcd", [0, 1])
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", SHAPES)
def test_decode_and_queue_do_not_see_stale_slots(dtype, d, ps, hq, hkv, per_xcd):
    """Decodes whose contexts end inside a group, at its end and inside a step; as a decode batch and as a queue beside a chunk."""
    g = I.Geometry(hq, hkv, d, ps, 6144 // ps + 64, dtype)
    prefix, new = [0, 15, 16, 37, 150, 700, 4000, 90], [1, 1, 1, 1, 1, 1, 1, 9]
    want = None
    with cus(per_xcd):
        for stale in (0.0, float("nan"), float("inf"), -float("inf")):
            bt = I.deal_block_tables(I.rng_for(84, 0), [p + n for p, n in zip(prefix, new)], ps, g.num_pages)
            cache = make_cache(g)
            cache.k_pool.fill_(stale)
            cache.v_pool.fill_(stale)
            fill, chunk = DevBatch(make_batch(g, [0] * 8, prefix, seed=84, bt=bt)), DevBatch(make_batch(g, prefix, new, seed=84, bt=bt, stream=2))
            for b in (fill, chunk):
                B.ag_kv_append(cache, b.k_new, b.v_new, b.bt, b.prefix, b.new, b.cu, b.total)
            got = [gpu_decode(cache, chunk.q[:8].contiguous(), chunk.bt, chunk.ctx, chunk.max_ctx, g), gpu_merged(cache, chunk),
                   gpu_merged(cache, chunk, own_kernel=True)]
            want = want or got
            for a, b in zip(got, want):
                assert (a == b).all(), f"stale slots of {stale}"
