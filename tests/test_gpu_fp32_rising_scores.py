"""fp32 prefill in tiles where the reference maximum of a column is outgrown in every tile, in none after the first, or by one head of
a wave's only: a wave then leaves the tile loop to rescale and enters it again, also in the tiles that straddle the diagonal."""
import numpy as np
import pytest

from gpu_helpers import DevBatch, gpu_append, gpu_prefill, make_cache
from helpers import fresh_pools, make_batch, oracle_append, oracle_attn
from paper_2603_10342_amd import inputs as I
from test_gpu_precision import cus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,lens", [(8, 2, [290, 33, 1, 160]), (6, 2, [129, 257]), (4, 4, [300, 127])])
def test_a_reference_maximum_that_is_outgrown_in_every_tile(hq, hkv, lens, d):
    g = I.Geometry(hq, hkv, d, 16, 64, I.F32)
    b = make_batch(g, [0] * len(lens), lens, seed=66)
    # scores rise by 8 (11.5 powers of two; 8 are let pass) a tile of 32 keys for every third head, fall for the next
    b.q[:, 0::3, 0], b.q[:, 1::3, 0], b.q[:, 2::3, 0] = 1.0, -1.0, 0.0
    at = np.concatenate([np.arange(n) for n in lens]).astype(np.float32)
    b.k_new[:, :, 0] = (0.25 * np.sqrt(d) * at)[:, None]
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    db = DevBatch(b)
    with cus(1):
        gpu_append(cache, db)
        got = gpu_prefill(cache, db)
    oracle_append(kp, vp, b)
    ref = oracle_attn(kp, vp, b)
    # the relative gate of fp32, and the exponent, up to 75 and in powers of two 109, rounded to 2^-18 three times
    gate = 1e-5 + 3 * 2.0 ** -18
    for h in range(hq):
        err, size = np.linalg.norm(got[:, h] - ref[:, h]), np.linalg.norm(ref[:, h])
        assert err <= gate * size, f"head {h}: {err:.2e} of {size:.2e}"
