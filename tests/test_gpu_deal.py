"""Prefill tiles dealt to the XCDs: every number of XCDs that share heads (1, 2, 4 and 8), lists that fit the chip at once and
lists that are dealt in runs (eight CUs), ragged chunks and prompts of one length, against the oracle."""
import pytest
import torch

from gpu_helpers import check_close, make_cache, run_phase
from helpers import fresh_pools, make_batch
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,ps", [(I.BF16, 128, 16), (I.BF16, 64, 32), (I.BF16, 256, 16), (I.F32, 64, 16), (I.F32, 128, 16)])
@pytest.mark.parametrize("hq,hkv", [(8, 8), (8, 4), (12, 2), (6, 6), (3, 1)])
@pytest.mark.parametrize("cus_per_xcd", [0, 1])
def test_every_tile_once(dtype, d, ps, hq, hkv, cus_per_xcd):
    g = I.Geometry(hq, hkv, d, ps, 4096 // ps, dtype)
    for prefix, new in (([0] * 4, [130] * 4), ([0, 300, 0, 40, 0, 7], [200, 3, 90, 41, 1, 160])):
        bt = I.deal_block_tables(I.rng_for(91, 0), [p + n for p, n in zip(prefix, new)], ps, g.num_pages)
        cache = make_cache(g)
        kp, vp = fresh_pools(g)
        stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, cus_per_xcd)) if cus_per_xcd else None
        try:
            torch.cuda.synchronize()
            with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.current_stream()):
                if any(prefix):
                    run_phase(cache, kp, vp, make_batch(g, [0] * len(prefix), prefix, seed=91, bt=bt, sigma_qk=1.0, sigma_v=1.0), "cold")
                got, ref = run_phase(cache, kp, vp, make_batch(g, prefix, new, seed=91, bt=bt, stream=2, sigma_qk=1.0, sigma_v=1.0), "resume")
        finally:
            torch.cuda.synchronize()
            if stream:
                B.ag_stream_destroy(stream)
        check_close(got, ref, dtype, f"{g} on {cus_per_xcd} CUs per XCD")
