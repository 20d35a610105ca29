"""Prefill of few rows at 256 channels (the keys of a query tile split over four waves) and both sides of the line between that
kernel and the others, which depends on the contexts: edges of steps, of the waves' shares, of tiles, against the oracle."""
import numpy as np
import pytest

from gpu_helpers import check_close, make_cache, run_phase
from helpers import fresh_pools, make_batch
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
