"""Which kernel a call takes, at batches where both sides of a line were measured and differ (the figures stand at the lines in
the sources): seen on the CPU, through a HIP runtime that logs launches."""
import pytest

from launches import launched


@pytest.fixture(scope="module")
def tmp(tmp_path_factory):
    return tmp_path_factory.mktemp("launches")


def kernels(tmp, *calls):
    return [[l.split(" ")[0] for l in r] for r in launched(calls, tmp)]


H82, H162 = dict(hq=8, hkv=2), dict(hq=16, hkv=2)


@pytest.mark.parametrize("page,columns,batches", [
    (16, 128, [dict(batch=1, new=2048), dict(batch=3, prefix=2000, new=700), dict(batch=16, new=1500), dict(batch=64, new=600), dict(batch=64, new=1500)]),
    (16, 256, [dict(batch=2, new=1000), dict(batch=2, prefix=2000, new=1000), dict(batch=4, prefix=3000, new=512), dict(batch=6, prefix=4000, new=1024, **H82),
               dict(batch=8, new=4096)]),
    (32, 128, [dict(batch=1, new=2048), dict(batch=3, prefix=2000, new=700), dict(batch=64, new=1000)]),
    (32, 256, [dict(batch=2, prefix=6000, new=600), dict(batch=1, prefix=3000, new=3000, **H162), dict(batch=6, prefix=4000, new=1024, **H82), dict(batch=2, prefix=2000, new=1000),
               dict(batch=4, new=2048)]),
])
def test_columns_of_a_prefill_workgroup(tmp, page, columns, batches):
    tail = "false,true" if page == 16 else "true,false"
    for b, k in zip(batches, kernels(tmp, *(dict(call="resume", page=page, **b) for b in batches))):
        assert k == [f"prefill_mfma_kernel<{columns // 32},128,{tail}>"], b


SPLIT = "prefill_split_kernel"


@pytest.mark.parametrize("shape,split,batches", [
    (dict(d=256), False, [dict(batch=29, prefix=274, new=101, **H82), dict(batch=21, prefix=25, new=13),
                          dict(batch=8, new=100), dict(batch=8, prefix=1500, new=160)]),
    (dict(d=256), True, [dict(batch=8, prefix=300, new=60), dict(batch=16, prefix=600, new=30), dict(batch=6, prefix=2200, new=13), dict(batch=44, prefix=21, new=7)]),
    (dict(dtype="f32"), False, [dict(batch=19, prefix=190, new=63, **H162), dict(batch=16, new=50), dict(batch=2, new=1000)]),
    (dict(dtype="f32"), True, [dict(batch=44, prefix=32, new=3), dict(batch=1, prefix=6000, new=211)]),
    (dict(d=64), False, [dict(batch=16, new=50), dict(batch=8, prefix=2000, new=100)]),
    (dict(d=64), True, [dict(batch=8, prefix=300, new=60), dict(batch=16, prefix=600, new=30)]),
    (dict(), False, [dict(batch=8, new=50), dict(batch=8, prefix=2000, new=100)]),
    (dict(), True, [dict(batch=5, new=60, **H162), dict(batch=1, prefix=6007, new=400)]),
])
def test_few_rows_or_whole_tiles(tmp, shape, split, batches):
    for b, k in zip(batches, kernels(tmp, *(dict(call="resume", **shape, **b) for b in batches))):
        assert len(k) == 1 and k[0].startswith(SPLIT) == split, (b, k)


F64, F128 = dict(dtype="f32", d=64), dict(dtype="f32")


@pytest.mark.parametrize("alone,batches", [
    (True, [dict(batch=1, max_ctx=850, hq=4, hkv=4, **F64), dict(batch=1, max_ctx=1770, d=64, **H82), dict(batch=1, max_ctx=440, **F128), dict(batch=1, max_ctx=440, d=256),
            dict(batch=30, max_ctx=2200, d=64), dict(batch=64, max_ctx=120, **F64)]),
    (False, [dict(batch=1, max_ctx=878, hq=4, hkv=4, **F64), dict(batch=1, max_ctx=1800, d=64, **H82), dict(batch=1, max_ctx=460, **F128), dict(batch=30, max_ctx=4200, d=64)]),
])
def test_decode_one_workgroup_a_pair_or_shares(tmp, alone, batches):
    for b, k in zip(batches, kernels(tmp, *(dict(call="decode", page=32, **b) for b in batches))):
        assert [x.split("<")[0] for x in k] == (["decode_any_direct_kernel"] if alone else ["decode_any_split_kernel", "decode_any_merge_kernel"]), b
