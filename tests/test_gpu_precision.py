"""What is computed in 32 bits stays in 32 bits: softmax weights of bf16 caches beside the bf16 / 128 / 16 shape (more than 16
heads a group included), and fp32 numbers so small that bf16 terms lose them.  Rows that are not finite are the row-by-row
kernel's bit for bit, and take no longer than there."""
import contextlib

import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_decode, gpu_merged, gpu_prefill, gpu_resume, make_cache
from helpers import fresh_pools, make_batch, oracle_append, oracle_attn
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def cus(per_xcd):
    """A stream of per_xcd CUs of every XCD (0: the whole device): small batches then count as many tiles and pairs."""
    stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, per_xcd)) if per_xcd else None
    try:
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
            yield
    finally:
        torch.cuda.synchronize()
        if stream:
            B.ag_stream_destroy(stream)


def two_opposite_keys(d, ps, hq, hkv, prefix, seed, batch=40):
    """Every session ends in two keys whose scores differ by 2^-11 to 2^-10 and whose values are +1 and -1, behind one whose
    score is 0.875 higher and whose value is 0, and `prefix` keys of no weight: the last row is the difference of two nearly
    equal weights of about 0.4, over their sum."""
    p, n = np.full(batch, prefix, np.int32), np.full(batch, 3, np.int32)
    pages = batch * ((prefix + 3 + ps - 1) // ps) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, I.BF16)
    rng = np.random.default_rng(seed)
    bt = I.deal_block_tables(I.rng_for(seed, 0), p + n, ps, pages)
    k, v = np.zeros((batch * prefix, hkv, d)), np.ones((batch * prefix, hkv, d))
    k[:, :, 2] = -4096.0
    fill = make_batch(g, np.zeros_like(p), p, seed=seed, bt=bt, k=k, v=v) if prefix else None
    k, v = np.zeros((3 * batch, hkv, d)), np.ones((3 * batch, hkv, d))
    k[:, :, 0] = 1.0
    k[0::3, :, 0], v[0::3] = 1.875, 0.0
    k[2::3, :, 1] = -rng.uniform(2.0 ** -8, 2.0 ** -7, size=(batch, hkv))
    v[2::3] = -1.0
    q = np.zeros((3 * batch, hq, d))
    q[:, :, 0] = q[:, :, 2] = 8.0
    q[:, :, 1] = 1.0
    return g, fill, make_batch(g, p, n, seed=seed, bt=bt, q=q, k=k, v=v, stream=2), 0.125


# A relative error e of one weight is e 2^10 to e 2^11 of the result.  Allowed: the result's own rounding to bf16, 2^-8 (eight
# significant bits), and 2^-10 for fp32 arithmetic (scores, exponentials and sums: a few 2^-24 of the weights, up to 2^-11 of
# the result).  Weights as two bf16 terms are off by up to 2^-17 each, up to 2^-6 of the result.
LIMIT = 2.0 ** -8 + 2.0 ** -10


def check_difference(got, ref, what):
    err = np.abs(got - ref) / np.abs(ref)
    assert err.max() <= LIMIT, f"{what}: {err.max():.2e} of the result"


@pytest.mark.parametrize("cus_per_xcd", [0, 1])
@pytest.mark.parametrize("prefix", [0, 70])
@pytest.mark.parametrize("d,ps,hq,hkv", [(64, 64, 8, 2), (64, 16, 4, 4), (128, 32, 8, 2), (72, 32, 5, 1), (256, 16, 6, 2), (128, 64, 40, 2)])
def test_bf16_caches_keep_their_softmax_weights_in_32_bits(d, ps, hq, hkv, prefix, cus_per_xcd):
    g, fill, b, scale = two_opposite_keys(d, ps, hq, hkv, prefix, seed=61)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    for x in (fill, b):
        if x is not None:
            gpu_append(cache, DevBatch(x))
            oracle_append(kp, vp, x)
    ref = oracle_attn(kp, vp, b, scale=scale)[2::3]
    db = DevBatch(b)
    with cus(cus_per_xcd):
        got = gpu_resume(cache, db, scale) if prefix else gpu_prefill(cache, db, scale)
        check_difference(got[2::3], ref, "prefill")
        check_difference(gpu_merged(cache, db, scale)[2::3], ref, "queue")
        got = gpu_decode(cache, db.q[2::3].contiguous(), db.bt, db.ctx, db.max_ctx, g, scale)
        check_difference(got, ref, "decode")


# bf16 / 128 / 16 with more query heads per KV head than the merged kernel's tiles hold: its queue, like its decode, keeps
# weights in 32 bits (ag_attn_prefill and ag_attn_resume round them at this shape).
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
@pytest.mark.parametrize("prefix", [0, 70])
def test_queues_of_large_groups_keep_their_softmax_weights_in_32_bits(prefix, cus_per_xcd):
    g, fill, b, scale = two_opposite_keys(128, 16, 40, 2, prefix, seed=62)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    for x in (fill, b):
        if x is not None:
            gpu_append(cache, DevBatch(x))
            oracle_append(kp, vp, x)
    ref = oracle_attn(kp, vp, b, scale=scale)[2::3]
    db = DevBatch(b)
    with cus(cus_per_xcd):
        check_difference(gpu_merged(cache, db, scale)[2::3], ref, "queue")
        got = gpu_decode(cache, db.q[2::3].contiguous(), db.bt, db.ctx, db.max_ctx, g, scale)
        check_difference(got, ref, "decode")


@pytest.mark.parametrize("cus_per_xcd", [0, 1])
def test_an_infinite_value_in_a_queue_of_large_groups_stays_with_the_rows_that_see_it(cus_per_xcd):
    lens, at, ch, G = [130, 143], 100, 67, 20
    g = I.Geometry(2 * G, 2, 128, 16, 24, I.BF16)
    bt = I.deal_block_tables(I.rng_for(63, 0), lens, 16, 24)
    b = make_batch(g, [0, 0], lens, seed=63, bt=bt)
    kp, vp = fresh_pools(g)
    oracle_append(kp, vp, b)
    ref = oracle_attn(kp, vp, b)
    cache, db = make_cache(g), DevBatch(b)
    db.v_new[at, 0, ch] = float("inf")
    gpu_append(cache, db)
    with cus(cus_per_xcd):
        got = gpu_merged(cache, db)
    assert np.all(got[at:lens[0], :G, ch] == np.inf)
    got[at:lens[0], :G, ch] = ref[at:lens[0], :G, ch]
    check_close(got, ref, I.BF16, "queue, 40 / 2 heads")


# fp32 prefill of many tiles takes numbers as three bf16 terms each, which lie up to 2^-16 below the number: what is too
# small for its terms has to be noticed, wherever it stands.  Every other value channel, every other key or query, or
# everything, is scaled down by `small`; the other side of a product is scaled up, so that scores stay as they are.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what,small", [("channels", 2.0 ** -120), ("channels", 2.0 ** -105), ("values", 2.0 ** -120), ("values", 2.0 ** -140),
                                        ("keys", 2.0 ** -122), ("queries", 2.0 ** -122), ("weights", 2.0 ** -122)])
def test_fp32_prefill_keeps_small_numbers_in_32_bits(what, small, d):
    lens = [150, 290]
    g = I.Geometry(8, 2, d, 16, 40, I.F32)
    b = make_batch(g, [0, 0], lens, seed=64)
    scaled = np.zeros((sum(lens), 1, d), bool)
    if what == "channels":
        scaled[:, :, 1::2] = True
    elif what == "values":
        scaled[:] = True
    if what in ("channels", "values"):
        b.v_new = (b.v_new * np.where(scaled, small, 1.0)).astype(np.float32)
        b.v_new[:, :, 7] = 0.0                                  # (a channel of zeros is no small number)
    elif what == "weights":
        # the first key outweighs the second by 1 / small and up to 8 times that, the others by far more, and only the second
        # one has values, large ones: the result is its small weight times those
        first = np.array([0, lens[0]])
        v = b.v_new[first + 1] * np.float32(2.0 ** 60)
        b.v_new[:], b.q[:], b.k_new[:] = 0.0, 0.0, 0.0
        b.v_new[first + 1] = v
        b.q[:, :, 0] = np.random.default_rng(64).uniform(1.0, 1.0 - np.log(8.0) / np.log(small), size=b.q.shape[:2])
        b.k_new[:, :, 0] = 2.0 * np.log(small) * np.sqrt(d)
        b.k_new[first, :, 0], b.k_new[first + 1, :, 0] = 0.0, np.log(small) * np.sqrt(d)
    else:
        down, up = (b.k_new, b.q) if what == "keys" else (b.q, b.k_new)
        down *= np.float32(small)
        up *= np.float32(1.0 / small)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    db = DevBatch(b)
    with cus(1):
        gpu_append(cache, db)
        got = gpu_prefill(cache, db)
    oracle_append(kp, vp, b)
    ref = oracle_attn(kp, vp, b)
    # per channel, so that none hides behind larger ones: the relative gate of fp32, and half a unit of the smallest number
    # for every term of a sum whose result is as small.  Weights: the exponent of about 85 is rounded to 2^-18 three times
    # (product, scaled score, difference).
    gate = 1e-5 + (3 * 2.0 ** -18 if what == "weights" else 0.0)
    for ch in range(d):
        err, size = np.linalg.norm(got[:, :, ch] - ref[:, :, ch]), np.linalg.norm(ref[:, :, ch])
        least = 2.0 ** -150 * np.sqrt(sum(lens) * 8) * max(lens)
        assert err <= gate * size + least, f"channel {ch}: {err:.2e} of {size:.2e}"


def off_16_bytes(t):
    """A copy whose address is no multiple of 16: such calls run row by row in plain fp32."""
    x = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:].view(t.shape)
    x.copy_(t)
    assert x.data_ptr() % 16
    return x


# Rows that are not finite are taken again in plain arithmetic: bit for bit what the row-by-row kernel gives, whichever
# rows share the pass, and the same every time.  head_dim 72 and 200: a merge workgroup's waves would hold parts of a row.
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [(I.BF16, 64, 64, 8, 2), (I.BF16, 128, 32, 8, 2), (I.BF16, 72, 16, 7, 1), (I.BF16, 200, 32, 6, 2),
                                               (I.BF16, 256, 16, 40, 2), (I.F32, 64, 16, 8, 2), (I.F32, 128, 256, 4, 4), (I.F32, 72, 32, 5, 1),
                                               (I.F32, 256, 16, 17, 1)])
def test_rows_taken_again_are_the_row_by_row_kernels(dtype, d, ps, hq, hkv, cus_per_xcd, bad):
    lens = [150, 290, 1]
    ctx = [n + 700 for n in lens]
    pages = sum((c + ps - 1) // ps for c in ctx) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(65, 0), ctx, ps, pages)
    fill = make_batch(g, [0] * 3, [700] * 3, seed=65, bt=bt)
    b = make_batch(g, [700] * 3, lens, seed=65, bt=bt, stream=2)
    cache, df, db = make_cache(g), DevBatch(fill), DevBatch(b)
    db.v_new[100, 0, 3] = bad                              # session 0: rows before and after it
    df.v_new[700 + 5, hkv - 1, d - 1] = bad                # session 1: every row
    gpu_append(cache, df)
    gpu_append(cache, db)
    last = torch.tensor([149, 439, 440], device="cuda")

    def run(q):
        db.q, db.out = q, torch.zeros_like(q)
        out = gpu_resume(cache, db)
        return out, gpu_decode(cache, q[last].contiguous() if q.data_ptr() % 16 == 0 else off_16_bytes(q[last]), db.bt, db.ctx, db.max_ctx, g)

    q = db.q
    with cus(cus_per_xcd):
        one, two = run(q), run(q)
    db.q = off_16_bytes(q)
    db.out = off_16_bytes(torch.zeros_like(q))
    rows = run(db.q)
    for x, again, want in zip(one, two, rows):
        assert np.array_equal(x, again, equal_nan=True)
        odd = ~np.isfinite(want).all(axis=-1)              # (row, head)
        assert odd.any() and not odd.all()
        np.testing.assert_array_equal(x[odd], want[odd])
        assert np.isfinite(x[~odd]).all()


@pytest.mark.parametrize("dtype,d,ps", [(I.BF16, 64, 64), (I.F32, 128, 16)])
def test_a_batch_with_a_value_that_is_not_finite_is_no_slower_than_row_by_row(dtype, d, ps):
    """Eight chunks on cached tokens, and a decode step, one session of which holds a NaN every row of it sees: against the
    same calls on a q off 16 bytes, which run row by row throughout (measured 4 times as long; one row after another in one
    wave, as it was, half as long)."""
    p, n = np.full(8, 1500, np.int32), np.full(8, 120, np.int32)
    g = I.Geometry(32, 8, d, ps, 8 * ((1620 + ps - 1) // ps), dtype)
    bt = I.deal_block_tables(I.rng_for(66, 0), p + n, ps, g.num_pages)
    fill, b = make_batch(g, np.zeros_like(p), p, seed=66, bt=bt), make_batch(g, p, n, seed=66, bt=bt, stream=2)
    cache, df, db = make_cache(g), DevBatch(fill), DevBatch(b)
    df.v_new[1, 0, 3] = float("nan")
    gpu_append(cache, df)
    gpu_append(cache, db)

    def shortest(call):
        call()
        times = []
        for _ in range(3):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    ws = torch.empty(B.ag_attn_decode_workspace_bytes(8, 32, d, db.max_ctx) // 4, dtype=torch.float32, device="cuda")
    last = torch.arange(8, device="cuda") * 120 + 119
    q, q1 = db.q, db.q[last].contiguous()
    out, out1 = torch.empty_like(q), torch.empty_like(q1)
    for q_, o_, q1_, o1_ in ((q, out, q1, out1), (off_16_bytes(q), off_16_bytes(out), off_16_bytes(q1), off_16_bytes(out1))):
        t = (shortest(lambda: B.ag_attn_resume(cache, q_, o_, db.bt, db.prefix, db.new, db.cu, db.total, db.max_new, db.max_ctx, 32, g.scale)),
             shortest(lambda: B.ag_attn_decode(cache, q1_, o1_, db.bt, db.ctx, db.max_ctx, 32, g.scale, ws)))
        if q_ is q:
            mended = t
    assert mended[0] <= t[0] and mended[1] <= t[1], (mended, t)
