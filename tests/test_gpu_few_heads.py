"""fp32 decode with at most four query heads a KV head runs on 4x4x1 products in sub-steps of 32 tokens: every number of
heads, contexts around the sub-steps, chunks and shares, both ways of dealing the work, against the fp64 oracle."""
import numpy as np
import pytest

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_decode, i32, make_cache, to_dev
from helpers import fresh_pools, make_batch, oracle_append
from oracle import oracle as O
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu

CTX = np.array([1, 3, 4, 5, 8, 9, 15, 16, 17, 24, 31, 32, 33, 0, 63, 64, 65, 257, 290, 511, 800], np.int32)


@pytest.mark.parametrize("d,ps", [(64, 16), (64, 128), (128, 16), (128, 32)])
@pytest.mark.parametrize("hq,hkv", [(1, 1), (2, 1), (6, 2), (4, 1)])
def test_decode_around_sub_steps(d, ps, hq, hkv):
    """One workgroup a pair, then shares (by a bound far above the lengths); slots behind the last token hold NaN."""
    pages = int(sum((max(int(c), 1) + ps - 1) // ps for c in CTX)) + 3
    g = I.Geometry(hq, hkv, d, ps, pages, I.F32)
    bt = I.deal_block_tables(I.rng_for(71, 0), np.maximum(CTX, 1), ps, pages)
    fill = make_batch(g, np.zeros_like(CTX), CTX, seed=71, bt=bt, sigma_qk=1.0, sigma_v=1.0)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    df = DevBatch(fill)
    gpu_append(cache, df)
    oracle_append(kp, vp, fill)
    qn = I.normal_values(71, 9, 0, (len(CTX), hq, d), 1.0, I.F32)
    live = np.nonzero(CTX > 0)[0]
    ref = O.decode(kp, vp, I.F32, qn[live], bt[live], CTX[live], hq, g.scale)
    wide = np.concatenate([bt, np.zeros((len(CTX), 8000 // ps), np.int32)], axis=1)
    for table, bound in ((bt, int(CTX.max())), (wide, 8000)):
        got = gpu_decode(cache, to_dev(qn, I.F32), i32(table), i32(CTX), bound, g)
        assert np.all(got[CTX == 0] == 0)
        check_close(got[live], ref, I.F32, f"decode D={d} page={ps} {hq}/{hkv} bound {bound}")
