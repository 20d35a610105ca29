"""GPU parity of the kernels for every geometry beside bf16 / head_dim 128 / 16-token pages, against the fp64 oracle:
head dimensions at, below and between the sizes the kernels are compiled for, pages of 16 to 256 tokens, groups of one
to more than 16 query heads, fp32 and bf16, contexts around the group, step and share boundaries."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_decode, gpu_merged, gpu_prefill, i32, make_cache, pools_match, run_phase, to_dev, to_f64
from helpers import fresh_pools, make_batch, oracle_append, oracle_attn
from oracle import oracle as O
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu

GEOMETRIES = [  # dtype, D, page, hq, hkv
    (I.BF16, 64, 16, 8, 2), (I.BF16, 64, 256, 4, 4), (I.BF16, 128, 32, 8, 2), (I.BF16, 256, 64, 6, 2), (I.BF16, 8, 16, 4, 2),
    (I.BF16, 72, 32, 16, 1), (I.BF16, 200, 16, 3, 1), (I.BF16, 128, 16, 40, 2), (I.F32, 64, 16, 8, 2), (I.F32, 128, 64, 4, 4),
    (I.F32, 256, 16, 6, 2), (I.F32, 24, 128, 5, 1), (I.F32, 136, 32, 17, 1), (I.F32, 128, 16, 32, 8)]


@pytest.mark.parametrize("dtype,d,ps,hq,hkv", GEOMETRIES)
def test_decode_boundary_lengths(dtype, d, ps, hq, hkv):
    """One token up to several shares; slots behind the last token and unused pages hold NaN."""
    ctx = np.array([1, 15, 16, 17, 0, 31, 32, 33, 48, 127, 129, 255, 257, 513, 1100], np.int32)
    pages = int(sum((max(int(c), 1) + ps - 1) // ps for c in ctx)) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(51, 0), np.maximum(ctx, 1), ps, pages)
    fill = make_batch(g, np.zeros_like(ctx), ctx, seed=51, bt=bt, sigma_qk=1.0, sigma_v=1.0)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    d_fill = DevBatch(fill)
    gpu_append(cache, d_fill)
    oracle_append(kp, vp, fill)
    qn = I.normal_values(51, 9, 0, (len(ctx), hq, d), 1.0, dtype)
    got = gpu_decode(cache, to_dev(qn, dtype), d_fill.bt, i32(ctx), int(ctx.max()), g)
    live = np.nonzero(ctx > 0)[0]
    assert np.all(got[ctx == 0] == 0)
    ref = O.decode(kp, vp, dtype, qn[live], bt[live], ctx[live], hq, g.scale)
    check_close(got[live], ref, dtype, f"decode D={d} page={ps} {hq}/{hkv}")


@pytest.mark.parametrize("dtype,d", [(I.BF16, 64), (I.F32, 128)])
def test_decode_shares_that_span_many_short_sessions(dtype, d):
    """More sessions than one pass of the plan covers, some empty; then a bound far above the lengths."""
    g = I.Geometry(8, 2, d, 32, 1500, dtype)
    rng = np.random.default_rng(52)
    ctx = rng.integers(1, 130, size=300).astype(np.int32)
    ctx[rng.integers(0, 300, size=40)] = 0
    ctx[[0, 255, 256, 299]] = [0, 33, 0, 1]
    bt = I.deal_block_tables(I.rng_for(52, 0), np.maximum(ctx, 1), 32, g.num_pages)
    fill = make_batch(g, np.zeros_like(ctx), ctx, seed=52, bt=bt, sigma_qk=1.0, sigma_v=1.0)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    d_fill = DevBatch(fill)
    gpu_append(cache, d_fill)
    oracle_append(kp, vp, fill)
    qn = I.normal_values(52, 9, 0, (300, 8, d), 1.0, dtype)
    live = np.nonzero(ctx > 0)[0]
    ref = O.decode(kp, vp, dtype, qn[live], bt[live], ctx[live], 8, g.scale)
    wide = np.concatenate([bt, np.zeros((300, 600), np.int32)], axis=1)
    for table, bound in ((bt, int(ctx.max())), (wide, 16000)):
        got = gpu_decode(cache, to_dev(qn, dtype), i32(table), i32(ctx), bound, g)
        assert np.all(got[ctx == 0] == 0)
        check_close(got[live], ref, dtype, f"decode, 300 sessions, bound {bound}")


@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [(I.BF16, 128, 16, 8, 2), (I.BF16, 128, 16, 16, 1), (I.BF16, 64, 32, 8, 2),
                                               (I.BF16, 256, 16, 6, 2), (I.F32, 64, 16, 40, 2), (I.F32, 128, 16, 8, 2), (I.F32, 64, 16, 4, 1)])
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
def test_decode_at_the_line_between_one_workgroup_per_pair_and_shares(dtype, d, ps, hq, hkv, cus_per_xcd):
    """max_ctx at and one past the most that one workgroup goes through alone: 416 KiB of keys and values a pair for bf16 / 128 / 16, 432 of
    fp32 at 64 channels, 448 of the others, on the whole device; 512 KiB and 1 MiB on 8 CUs where the six pairs of one KV head are over
    half of them (more never get one each).  Lengths from one token to the bound, some empty.  bf16 / 128 / 16: the step in one
    launch as well, with the same bits on either side."""
    main = (dtype, d, ps) == (I.BF16, 128, 16)
    if cus_per_xcd and hkv == 1:
        kib = 512 if main else 1024
    else:
        kib = 416 if main else 432 if (dtype, d) == (I.F32, 64) else 448
    line = (kib << 10) // (2 * d * (4 if dtype == I.F32 else 2))
    stream = None
    if cus_per_xcd:
        stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, cus_per_xcd))
    try:
        for top in (line, line + 1):
            ctx = np.array([top, 0, 1, 33, top // 2 + 5, top - 1], np.int32)
            pages = int(sum((max(int(c), 1) + ps - 1) // ps for c in ctx)) + 3
            g = I.Geometry(hq, hkv, d, ps, pages, dtype)
            bt = I.deal_block_tables(I.rng_for(57, 0), np.maximum(ctx, 1), ps, pages)
            fill = make_batch(g, np.zeros_like(ctx), ctx, seed=57, bt=bt)
            cache = make_cache(g)
            kp, vp = fresh_pools(g)
            df = DevBatch(fill)
            gpu_append(cache, df)
            oracle_append(kp, vp, fill)
            qn = I.normal_values(57, 9, 0, (len(ctx), hq, d), 1.0, dtype)
            live = np.nonzero(ctx > 0)[0]
            ref = O.decode(kp, vp, dtype, qn[live], bt[live], ctx[live], hq, g.scale)
            torch.cuda.synchronize()
            with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
                got = gpu_decode(cache, to_dev(qn, dtype), df.bt, i32(ctx), top, g)
            assert np.all(got[ctx == 0] == 0)
            check_close(got[live], ref, dtype, f"decode up to {top} D={d} {hq}/{hkv}")
            if main:
                last = [int(fill.cu_new[i + 1]) - 1 for i in range(len(ctx))]          # a session's newest token, taken again
                k, v = (to_dev(x[last], dtype) for x in (fill.k_new, fill.v_new))
                q, ws = to_dev(qn, dtype), torch.zeros(B.ag_decode_step_workspace_bytes(len(ctx), hq, d, top) // 4, dtype=torch.float32, device="cuda")
                out = torch.full_like(q, float("nan"))
                torch.cuda.synchronize()
                B.ag_decode_step(cache, k, v, q, out, df.bt, i32(ctx), top, hq, g.scale, ws, stream=stream)
                torch.cuda.synchronize()
                assert np.array_equal(to_f64(out, dtype), got)
                pools_match(cache, kp, vp, dtype)
    finally:
        torch.cuda.synchronize()
        if stream:
            B.ag_stream_destroy(stream)


def test_decode_of_a_q_that_is_not_16_byte_aligned_still_runs():
    g = I.Geometry(3, 1, 24, 16, 8, I.F32)
    ctx = np.array([40, 7], np.int32)
    bt = I.deal_block_tables(I.rng_for(53, 0), ctx, 16, 8)
    fill = make_batch(g, [0, 0], ctx, seed=53, bt=bt, sigma_qk=1.0, sigma_v=1.0)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    d_fill = DevBatch(fill)
    gpu_append(cache, d_fill)
    oracle_append(kp, vp, fill)
    qn = I.normal_values(53, 9, 0, (2, 3, 24), 1.0, I.F32)
    buf = torch.empty(2 * 3 * 24 + 1, dtype=torch.float32, device="cuda")
    q = buf[1:].view(2, 3, 24)
    q.copy_(torch.from_numpy(qn))
    assert q.data_ptr() % 16
    got = gpu_decode(cache, q, d_fill.bt, i32(ctx), 40, g)
    check_close(got, O.decode(kp, vp, I.F32, qn, bt, ctx, 3, g.scale), I.F32, "decode, unaligned q")


@pytest.mark.parametrize("dtype,d,ps,hq,hkv", GEOMETRIES)
def test_cold_then_resume_around_tile_edges(dtype, d, ps, hq, hkv):
    """Chunks around the 32- and 64-key tiles and the 128-column workgroups, an empty one, ragged prefixes; NaN behind
    every context."""
    lens_a, lens_b = [33, 0, 64, 1, 150, 16], [31, 40, 65, 130, 5, 0]
    pages = sum((a + b + ps - 1) // ps for a, b in zip(lens_a, lens_b)) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(54, 0), [a + b for a, b in zip(lens_a, lens_b)], ps, pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    cold = make_batch(g, [0] * 6, lens_a, seed=54, bt=bt)
    got, ref = run_phase(cache, kp, vp, cold, "cold")
    check_close(got, ref, dtype, f"cold D={d} page={ps} {hq}/{hkv}")
    more = make_batch(g, lens_a, lens_b, seed=54, bt=bt, stream=2)
    got, ref = run_phase(cache, kp, vp, more, "resume")
    check_close(got, ref, dtype, f"resume D={d} page={ps} {hq}/{hkv}")
    pools_match(cache, kp, vp, dtype)


# Query tiles that do not fill the chip take a kernel that splits the keys over a workgroup's waves (head_dim 64 and
# 128; every call of the tests above, and of the small tests of the bf16 / 128 / 16 shape); on a stream of 8 CUs the same
# calls count as many tiles and take the kernels that the whole device uses for large batches.
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [GEOMETRIES[i] for i in (0, 1, 2, 7, 8, 9, 13)] + [
    (I.BF16, 128, 16, 8, 2), (I.BF16, 128, 16, 3, 1), (I.BF16, 128, 16, 4, 2), (I.BF16, 128, 16, 8, 1)])
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
def test_split_and_whole_tiles_agree_with_the_oracle(dtype, d, ps, hq, hkv, cus_per_xcd):
    lens_a, lens_b = [33, 0, 600, 1, 150, 290], [31, 40, 65, 530, 5, 0]
    pages = sum((a + b + ps - 1) // ps for a, b in zip(lens_a, lens_b)) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(56, 0), [a + b for a, b in zip(lens_a, lens_b)], ps, pages)
    kp, vp = fresh_pools(g)
    cold = make_batch(g, [0] * 6, lens_a, seed=56, bt=bt)
    more = make_batch(g, lens_a, lens_b, seed=56, bt=bt, stream=2)
    stream = None
    if cus_per_xcd:
        info = B.ag_device_info()
        stream = B.ag_stream_create_cumask(B.ag_cumask_build(info["num_cus"], 8, 0, cus_per_xcd))
    try:
        cache = make_cache(g)
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
            for b, kind in ((cold, "cold"), (more, "resume")):
                got, ref = run_phase(cache, kp, vp, b, kind)
                check_close(got, ref, dtype, f"{kind} D={d} page={ps} {hq}/{hkv} on {cus_per_xcd} CUs per XCD")
    finally:
        torch.cuda.synchronize()
        if stream:
            B.ag_stream_destroy(stream)


@pytest.mark.parametrize("dtype,d,ps", [(I.BF16, 64, 32), (I.F32, 128, 16)])
def test_merged_queue_and_sharp_logits(dtype, d, ps):
    """150 sessions, many without rows, with logits of standard deviation 4 (the reference maximum moves).  Queries and
    keys of sigma 2 each: an fp32 score of 128 such products is off by about sqrt(128) 2^-24 times the sum of its terms'
    sizes over sqrt(D), 29 here - a few 1e-6 in a weight, inside the 1e-5 gate, where sigma 4 (sum 115) would not be."""
    rng = np.random.default_rng(55)
    p, n = rng.integers(0, 101, size=150), rng.integers(0, 41, size=150)
    n[rng.integers(0, 150, size=30)] = 0
    n[[0, 63, 64, 127, 128, 149]] = [0, 40, 0, 1, 33, 0]
    pages = int(sum((int(a + b) + ps - 1) // ps for a, b in zip(p, n))) + 40
    g = I.Geometry(8, 2, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(55, 0), np.maximum(p + n, 1), ps, g.num_pages)
    fill = make_batch(g, np.zeros_like(p), p, seed=55, bt=bt)
    chunk = make_batch(g, p, n, seed=55, bt=bt, stream=2, sigma_qk=2.0)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    for b in (fill, chunk):
        gpu_append(cache, DevBatch(b))
        oracle_append(kp, vp, b)
    got, ref = gpu_merged(cache, DevBatch(chunk)), oracle_attn(kp, vp, chunk)
    check_close(got, ref, dtype, f"queue D={d} page={ps}")


# An infinity among the values belongs to the rows that see its token, and only to its channel; an infinite key makes the
# rows that see it infinite or leaves it out, by the sign of the query's channel.
@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [GEOMETRIES[i] for i in (0, 2, 3, 5, 6, 8, 9, 10, 11, 13)])
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
def test_an_infinite_value_stays_with_the_rows_that_see_it(dtype, d, ps, hq, hkv, cus_per_xcd):
    lens, at, ch, G = [150, 290], 100, d // 2 + 3, hq // hkv
    pages = sum((n + 1 + ps - 1) // ps for n in lens) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, dtype)
    bt = I.deal_block_tables(I.rng_for(58, 0), [n + 1 for n in lens], ps, pages)
    b = make_batch(g, [0, 0], lens, seed=58, bt=bt)
    one = make_batch(g, lens, [1, 1], seed=58, bt=bt, stream=2)
    kp, vp = fresh_pools(g)
    oracle_append(kp, vp, b)
    ref = oracle_attn(kp, vp, b)
    oracle_append(kp, vp, one)
    ref_one = oracle_attn(kp, vp, one)
    cache, db, d1 = make_cache(g), DevBatch(b), DevBatch(one)
    db.v_new[at, 0, ch] = float("inf")                     # session 0, token 100
    db.k_new[lens[0] + at, hkv - 1, ch] = float("-inf")    # session 1, token 100
    stream = None
    if cus_per_xcd:
        stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, cus_per_xcd))
    try:
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
            gpu_append(cache, db)
            got = gpu_prefill(cache, db)
            gpu_append(cache, d1)
            got_one = gpu_decode(cache, d1.q, d1.bt, d1.ctx, d1.max_ctx, g)
    finally:
        torch.cuda.synchronize()
        if stream:
            B.ag_stream_destroy(stream)
    for x, r, q, first, last, second in ((got, ref, b.q, at, lens[0], lens[0] + at), (got_one, ref_one, one.q, 0, 1, 1)):
        assert np.all(x[first:last, :G, ch] == np.inf)
        x[first:last, :G, ch] = r[first:last, :G, ch]
        seen, want = x[second:, (hkv - 1) * G:], r[second:, (hkv - 1) * G:]
        plus = I.stored_to_f64(q, dtype)[second:, (hkv - 1) * G:, ch] > 0        # score -inf: a weight of zero
        assert np.isfinite(seen[plus]).all() and np.isnan(seen[~plus]).all()
        seen[...] = want
        check_close(x, r, dtype, f"D={d} page={ps} {hq}/{hkv} on {cus_per_xcd} CUs per XCD")


@pytest.mark.parametrize("sigma_v", [1e-36, 1e-33, 1e37])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_keeps_its_precision_at_the_ends_of_its_range(d, sigma_v):
    """fp32 numbers taken as three bf16 terms (many columns per CU): the terms of tiny values leave the products' range."""
    g = I.Geometry(8, 2, d, 16, 40, I.F32)
    b = make_batch(g, [0, 0], [150, 290], seed=59, sigma_v=sigma_v)
    stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, 1))
    try:
        cache = make_cache(g)
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.ExternalStream(stream)):
            got, ref = run_phase(cache, *fresh_pools(g), b, "cold")
    finally:
        torch.cuda.synchronize()
        B.ag_stream_destroy(stream)
    check_close(got / sigma_v, ref / sigma_v, I.F32, f"cold D={d}, values of {sigma_v}")
