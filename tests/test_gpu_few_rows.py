"""Prefill of few rows at 256 channels (the keys of a query tile split over four waves) and both sides of the line between that
kernel and the others, which depends on the contexts; decode at the lines between one workgroup a pair and shares of the other
shapes: edges of steps, of the waves' shares, of tiles, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_decode, i32, make_cache, run_phase, to_dev
from helpers import fresh_pools, make_batch, oracle_append
from oracle import oracle as O
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


def fill_and_resume(g, prefix, new, seed):
    prefix, new = np.asarray(prefix, np.int32), np.asarray(new, np.int32)
    bt = I.deal_block_tables(I.rng_for(seed, 0), prefix + new, g.page_size, g.num_pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    if prefix.any():
        run_phase(cache, kp, vp, make_batch(g, np.zeros_like(prefix), prefix, seed=seed, bt=bt, sigma_qk=1.0, sigma_v=1.0), "cold")
    got, ref = run_phase(cache, kp, vp, make_batch(g, prefix, new, seed=seed, bt=bt, stream=2, sigma_qk=1.0, sigma_v=1.0), "resume")
    check_close(got, ref, g.dtype, f"{g}")


@pytest.mark.parametrize("ps,hq,hkv", [(16, 6, 2), (64, 4, 4), (32, 40, 2)])
def test_256_channels(ps, hq, hkv):
    g = I.Geometry(hq, hkv, 256, ps, 8192 // ps, I.BF16)
    # a wave's first, second and 33rd step (its page ids are fetched for 32 at a time), contexts that end inside a group,
    # rows that end a tile of 32 columns and do not
    fill_and_resume(g, [0, 31, 95, 127, 128, 500, 1, 4200], [1, 1, 33, 8, 9, 16, 40, 5], seed=61)


@pytest.mark.parametrize("dtype,d,ps", [(I.BF16, 128, 16), (I.BF16, 64, 32), (I.F32, 64, 16), (I.F32, 128, 16), (I.BF16, 256, 16)])
@pytest.mark.parametrize("sessions,rows,prefix", [(9, 13, 0), (9, 13, 700), (16, 50, 0)])
def test_around_the_line(dtype, d, ps, sessions, rows, prefix):
    g = I.Geometry(32, 8, d, ps, 1024, dtype)
    fill_and_resume(g, [prefix] * sessions, [rows - s % 3 for s in range(sessions)], seed=62)


@pytest.mark.parametrize("dtype,d,ps,hq,hkv", [(I.BF16, 64, 32, 8, 2), (I.BF16, 256, 16, 6, 2), (I.F32, 64, 16, 16, 1), (I.F32, 72, 32, 4, 2)])
@pytest.mark.parametrize("kib,cus_per_xcd", [(432, 0), (448, 0), (1024, 1)])
def test_decode_at_the_lines_of_one_workgroup_a_pair(dtype, d, ps, hq, hkv, kib, cus_per_xcd):
    """max_ctx at and one past what one workgroup goes through alone: 432 or 448 KiB, and 1 MiB where the pairs take more than half of the
    CUs (six or three on 8)."""
    padded = 64 if d <= 64 else 128 if d <= 128 else 256
    line = (kib << 10) // (2 * padded * (4 if dtype == I.F32 else 2))
    stream = None
    if cus_per_xcd:
        stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, cus_per_xcd))
    try:
        ctx = np.array([line, 0, line // 3 + 7] + ([17, 1, 16] if hkv == 1 else []), np.int32)
        pages = int(sum((int(c) + 2 + ps - 1) // ps for c in ctx)) + 3
        g = I.Geometry(hq, hkv, d, ps, pages, dtype)
        for extra in (0, 1):
            now = ctx + np.array([extra] + [0] * (len(ctx) - 1), np.int32)
            bt = I.deal_block_tables(I.rng_for(63, 0), np.maximum(now, 1), ps, pages)
            fill = make_batch(g, np.zeros_like(now), now, seed=63, bt=bt)
            cache = make_cache(g)
            kp, vp = fresh_pools(g)
            df = DevBatch(fill)
            gpu_append(cache, df)
            oracle_append(kp, vp, fill)
            qn = I.normal_values(63, 9, 0, (len(now), hq, d), 1.0, dtype)
            live = np.nonzero(now > 0)[0]
            ref = O.decode(kp, vp, dtype, qn[live], bt[live], now[live], hq, g.scale)
            torch.cuda.synchronize()
            with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
                got = gpu_decode(cache, to_dev(qn, dtype), df.bt, i32(now), int(now.max()), g)
            assert np.all(got[now == 0] == 0)
            check_close(got[live], ref, dtype, f"decode up to {now.max()} D={d} {hq}/{hkv}")
    finally:
        torch.cuda.synchronize()
        if stream:
            B.ag_stream_destroy(stream)
