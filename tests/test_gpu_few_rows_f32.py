"""fp32 prefill of few rows, whose products are of three bf16 terms: edges of its steps of 32 keys, of the eight waves' rounds (256
keys), of the 32 steps that a wave's page ids last for (8192 keys) and of its tiles of 32 columns; numbers whose terms leave the products' range, against the fp64 oracle within fp32's own gates."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_resume, make_cache, run_phase
from helpers import fresh_pools, make_batch, oracle_append, oracle_attn
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


def fill_and_resume(g, prefix, new, seed, sigma_qk=1.0, sigma_v=1.0):
    prefix, new = np.asarray(prefix, np.int32), np.asarray(new, np.int32)
    bt = I.deal_block_tables(I.rng_for(seed, 0), prefix + new, g.page_size, g.num_pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    if prefix.any():
        run_phase(cache, kp, vp, make_batch(g, np.zeros_like(prefix), prefix, seed=seed, bt=bt, sigma_qk=sigma_qk, sigma_v=sigma_v), "cold")
    got, ref = run_phase(cache, kp, vp, make_batch(g, prefix, new, seed=seed, bt=bt, stream=2, sigma_qk=sigma_qk, sigma_v=sigma_v), "resume")
    check_close(got / sigma_v, ref / sigma_v, g.dtype, f"{g}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("ps,hq,hkv", [(16, 6, 2), (64, 4, 4), (32, 40, 2), (128, 3, 1)])
def test_edges(d, ps, hq, hkv):
    g = I.Geometry(hq, hkv, d, ps, 8192 // ps, I.F32)
    fill_and_resume(g, [0, 31, 95, 127, 128, 500, 1, 4200], [1, 1, 33, 8, 9, 16, 40, 5], seed=61)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("ps,hq,hkv", [(16, 6, 2), (128, 3, 1)])
@pytest.mark.parametrize("prefix,new", [([254, 255, 256, 510, 511, 512], [1, 1, 1, 1, 2, 1]), ([8190, 8400], [3, 5])])
def test_ends_of_the_waves_rounds(d, ps, hq, hkv, prefix, new):
    """Contexts of 255, 256, 257, 511, 513 and 513 tokens, where a wave has one own step or two, or its second is the last one and partial;
    and of more than 8192, where it fetches page ids again."""
    g = I.Geometry(hq, hkv, d, ps, 20480 // ps, I.F32)
    fill_and_resume(g, prefix, new, seed=68)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sigma_qk,sigma_v", [(1.0, 1e-36), (1.0, 1e-33), (1.0, 1e37), (1e-15, 1.0)])
def test_ends_of_the_range(d, sigma_qk, sigma_v):
    g = I.Geometry(8, 2, d, 16, 64, I.F32)
    fill_and_resume(g, [0, 200], [45, 61], seed=64, sigma_qk=sigma_qk, sigma_v=sigma_v)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale_q,scale_k", [(1e-30, 1e30), (1e30, 1e-30), (1e25, 1e-26)])
def test_large_and_tiny_factors_of_ordinary_scores(d, scale_q, scale_k):
    g = I.Geometry(8, 2, d, 16, 64, I.F32)
    b = make_batch(g, [0, 0], [45, 61], seed=65, sigma_qk=1.0, sigma_v=1.0)
    b.q, b.k_new = (b.q * np.float32(scale_q)).astype(np.float32), (b.k_new * np.float32(scale_k)).astype(np.float32)
    got, ref = run_phase(make_cache(g), *fresh_pools(g), b, "cold")
    check_close(got, ref, I.F32, f"D={d} q {scale_q} k {scale_k}")


@pytest.mark.parametrize("d", [64, 128])
def test_zero_values_and_zero_keys(d):
    g = I.Geometry(8, 2, d, 16, 64, I.F32)
    b = make_batch(g, [0, 0], [45, 61], seed=66, sigma_qk=1.0, sigma_v=1.0)
    b.v_new[:, :, ::2] = 0
    b.k_new[:45] = 0
    got, ref = run_phase(make_cache(g), *fresh_pools(g), b, "cold")
    assert np.all(got[:, :, ::2] == 0)
    check_close(got, ref, I.F32, f"D={d}")


@pytest.mark.parametrize("d", [64, 128])
def test_zero_results_beside_values_below_the_terms_range(d):
    """Channels of zeros only, of values of 1e-38 that cancel to zero, and of values of 1e-33: the values are read again behind a result of
    zero, and the tile is taken once more where any of them is small."""
    g = I.Geometry(8, 2, d, 16, 64, I.F32)
    b = make_batch(g, [0, 0], [45, 300], seed=69, sigma_qk=1.0, sigma_v=1.0)
    b.v_new[:, :, 0] = 0
    b.v_new[:, 1, 3] *= np.float32(1e-33)
    b.v_new[:, 0, 5] = np.where(np.arange(345) % 2, np.float32(1e-38), np.float32(-1e-38))
    b.k_new[:, 0] = b.k_new[:1, 0]                              # KV head 0: equal weights, so that channel 5 cancels in every other row
    got, ref = run_phase(make_cache(g), *fresh_pools(g), b, "cold")
    assert np.all(got[:, :, 0] == 0)
    check_close(got, ref, I.F32, f"D={d}")
    check_close(got[:, 4:, 3] * 1e33, ref[:, 4:, 3] * 1e33, I.F32, f"D={d} channel 3")
    # a result has at most the rounding of its sums, of up to 300 numbers of 1e-38 that weigh 1 / 300 at least, and its own, of 2^-149
    assert np.abs(got[:, :4, 5] - ref[:, :4, 5]).max() <= 300 * 2.0 ** -24 * 1e-38 + 300 * 2.0 ** -149


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what", ["query", "value", "large value"])
def test_numbers_out_of_the_terms_range_on_a_long_context(d, what):
    """Five rows on 6000 tokens, a query channel of 1e-35 in one row, a value channel of 1e-33 or values of 2^80: taken with fp32
    products, at less than five times an ordinary call's time (row by row: eleven to sixteen times)."""
    g = I.Geometry(32, 8, d, 16, 400, I.F32)
    bt = I.deal_block_tables(I.rng_for(67, 0), [6005], 16, g.num_pages)
    first, b = (make_batch(g, [p], [n], seed=67, bt=bt, stream=i, sigma_qk=1.0, sigma_v=1.0) for i, (p, n) in enumerate([(0, 6000), (6000, 5)]))

    def timed(first, b):
        cache = make_cache(g)
        gpu_append(cache, DevBatch(first))
        df = DevBatch(b)
        gpu_append(cache, df)
        got, best = gpu_resume(cache, df), np.inf
        for _ in range(5):
            at = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            at[0].record()
            for _ in range(5):
                B.ag_attn_resume(cache, df.q, df.out, df.bt, df.prefix, df.new, df.cu, df.total, df.max_new, df.max_ctx, g.num_q_heads, g.scale)
            at[1].record()
            at[1].synchronize()
            best = min(best, at[0].elapsed_time(at[1]))
        return got, best

    _, usual = timed(first, b)
    size = 1.0
    if what == "query":
        b.q[2, 9, 5] = 1e-35
    elif what == "value":
        for x in (first, b):
            x.v_new[:, :, 7] *= np.float32(1e-33)
    else:
        size = 2.0 ** 80
        for x in (first, b):
            x.v_new *= np.float32(size)
    got, took = timed(first, b)
    kp, vp = fresh_pools(g)
    oracle_append(kp, vp, first)
    oracle_append(kp, vp, b)
    ref = oracle_attn(kp, vp, b)
    check_close(got / size, ref / size, I.F32, f"D={d} {what}")
    if what == "value":
        check_close(got[:, :, 7] * 1e33, ref[:, :, 7] * 1e33, I.F32, f"D={d} {what}, its channel")
    assert took < 5 * usual, (usual, took)
