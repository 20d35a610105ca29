"""Prefill tiles whose keys two sets of waves take in turn (few workgroups on long contexts; here on one CU per XCD): an even and an
odd number of key tiles, rows on both sides of a tile's end (the first one's too), ragged chunks; an infinite value in either set's tiles."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, check_close, gpu_append, gpu_resume, make_cache, run_phase
from helpers import fresh_pools, make_batch
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu


class few_cus:
    def __enter__(self):
        self.stream = B.ag_stream_create_cumask(B.ag_cumask_build(B.ag_device_info()["num_cus"], 8, 0, 1))
        torch.cuda.synchronize()
        self.scope = torch.cuda.stream(torch.cuda.ExternalStream(self.stream))
        self.scope.__enter__()

    def __exit__(self, *error):
        self.scope.__exit__(*error)
        torch.cuda.synchronize()
        B.ag_stream_destroy(self.stream)


SHAPES = [(128, 16), (128, 32), (64, 32), (64, 128)]
ACROSS = [(4, [37, 500], [100, 90]), (4, [61, 480], [40, 150]), (3, [61, 500], [100, 150]), (3, [1, 600], [135, 113])]      # query heads, prefixes, rows


@pytest.mark.parametrize("d,ps", SHAPES)
@pytest.mark.parametrize("prefix,new", [([262], [250]), ([326], [250]), ([390], [249]), ([1031], [250]), ([500, 0], [90, 130]), ([0, 777], [120, 100])])
def test_two_sets_of_waves(d, ps, prefix, new, hq=4):
    g = I.Geometry(hq, 1, d, ps, 4096 // ps, I.BF16)
    bt = I.deal_block_tables(I.rng_for(97, 0), [p + n for p, n in zip(prefix, new)], ps, g.num_pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    with few_cus():
        run_phase(cache, kp, vp, make_batch(g, [0] * len(prefix), prefix, seed=97, bt=bt, sigma_qk=1.0, sigma_v=1.0), "cold")
        got, ref = run_phase(cache, kp, vp, make_batch(g, prefix, new, seed=97, bt=bt, stream=2, sigma_qk=1.0, sigma_v=1.0), "resume")
    check_close(got, ref, I.BF16, f"{g} {prefix} {new}")


@pytest.mark.parametrize("d,ps", SHAPES)
@pytest.mark.parametrize("hq,prefix,new", ACROSS)
def test_rows_on_both_sides_of_the_first_key_tile(d, ps, hq, prefix, new):
    """Waves some of whose columns see no key of the second set's tiles, with 32 columns to a whole number of rows and (three heads a KV
    head) not."""
    test_two_sets_of_waves(d, ps, prefix, new, hq)


@pytest.mark.parametrize("d,ps", SHAPES)
@pytest.mark.parametrize("at", [10, 70, 300])
def test_an_infinite_value(d, ps, at):
    g = I.Geometry(4, 1, d, ps, 1024 // ps, I.BF16)
    bt = I.deal_block_tables(I.rng_for(98, 0), [600], ps, g.num_pages)
    cache = make_cache(g)
    kp, vp = fresh_pools(g)
    first, b = make_batch(g, [0], [350], seed=98, bt=bt), make_batch(g, [350], [250], seed=98, bt=bt, stream=2)
    with few_cus():
        run_phase(cache, kp, vp, first, "cold")
        want, ref = run_phase(cache, kp, vp, b, "resume")
        df = DevBatch(first)
        df.v_new[at, 0, 5] = float("inf")
        gpu_append(cache, df)
        got = gpu_resume(cache, DevBatch(b))
    assert np.all(got[:, :, 5] == np.inf)
    got[:, :, 5] = ref[:, :, 5]
    check_close(got, ref, I.BF16, f"{g} at {at}")
