"""The append of a decode's tokens - one a session, other slots of their pages in use or never written - with few and with many
workgroups, which store differently: pools bit for bit, nothing else touched."""
import numpy as np
import pytest

from gpu_helpers import DevBatch, gpu_append, make_cache, pools_match
from helpers import fresh_pools, make_batch, oracle_append
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [I.BF16, I.F32])
@pytest.mark.parametrize("d,ps", [(64, 16), (72, 32), (128, 64), (256, 16)])
@pytest.mark.parametrize("nb,hkv", [(1, 1), (31, 2), (32, 2), (21, 3), (70, 4)])      # 1, 62, 64, 63 and 280 workgroups
def test_one_token_a_session(dt, d, ps, nb, hkv):
    prefix = np.array([(0, 1, 7, 8, 15, 16, 17, 31, 63, 64)[i % 10] for i in range(nb)], np.int32)
    pages = int(sum((int(p) + ps) // ps for p in prefix)) + 3
    g = I.Geometry(hkv, hkv, d, ps, pages, dt)
    bt = I.deal_block_tables(I.rng_for(83, 0), prefix + 1, ps, pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    for b in (make_batch(g, np.zeros_like(prefix), prefix, seed=83, bt=bt, sigma_qk=1.0, sigma_v=1.0),
              make_batch(g, prefix, np.ones_like(prefix), seed=83, bt=bt, stream=2, sigma_qk=1.0, sigma_v=1.0)):
        if int(b.new_lens.sum()):
            gpu_append(cache, DevBatch(b))
            oracle_append(kp, vp, b)
    pools_match(cache, kp, vp, dt)
