"""Which kernel a call takes, at batches where both sides of a line were measured and differ (the figures stand at the lines in
the sources): seen on the CPU, through a HIP runtime that logs launches."""
import pytest

from launches import launched
from test_gpu_halves import ACROSS, SHAPES
from test_gpu_merged import FEW_ROWS, GROUPS, MIXES, SMALL


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


@pytest.mark.parametrize("alone,batches", [
    (True, [dict(batch=1, max_ctx=832), dict(batch=16, max_ctx=832), dict(batch=17, max_ctx=1024), dict(batch=32, max_ctx=1024), dict(batch=6, max_ctx=1024, hq=8, hkv=1, cus=8)]),
    (False, [dict(batch=1, max_ctx=833), dict(batch=16, max_ctx=833), dict(batch=17, max_ctx=1025), dict(batch=33, max_ctx=100), dict(batch=20, max_ctx=2048),
             dict(batch=6, max_ctx=1025, hq=8, hkv=1, cus=8), dict(batch=9, max_ctx=100, hq=8, hkv=1, cus=8)]),
])
def test_decode_and_step_of_the_main_shape(tmp, alone, batches):
    """One line for both, with more than half of the CUs busy and with fewer: their results are the same bits."""
    for b, k in zip(batches, kernels(tmp, *(dict(call="decode", **b) for b in batches))):
        assert [x.split("<")[0] for x in k] == (["decode_direct_kernel"] if alone else ["decode_split_kernel", "decode_merge_kernel"]), b
    for b, k in zip(batches, kernels(tmp, *(dict(call="step", **b) for b in batches))):
        assert [x.split("<")[0] for x in k] == ["decode_direct_kernel" if alone else "decode_split_kernel"], b


def queue(sessions, hq=8, hkv=2, **more):
    prefix, new = sessions
    return dict(call="merged", hq=hq, hkv=hkv, batch=len(new), total=sum(new), max_new=max(new), max_ctx=max(p + n for p, n in zip(prefix, new)), **more)


EXACT, MERGED, PREFILL = f"{SPLIT}<__bf16,128,false,true>", "merged_split_kernel", "prefill_"


def test_queues_of_the_gpu_tests_fall_on_the_sides_that_they_name(tmp):
    both = [MIXES[n] for n in ("empty_and_cold_like", "longest_kept", "only_resumes")] + [FEW_ROWS]
    want = [(queue(b, hq, hkv, cus=cus), EXACT if cus == 256 else MERGED) for b in both for hq, hkv in (GROUPS if b is FEW_ROWS else [(8, 2)]) for cus in (256, 8)]
    want += [(queue(MIXES[n], cus=cus), MERGED) for n in ("boundaries", "decodes_and_short_resumes") for cus in (256, 8)]
    want += [(queue(MIXES["handed_to_the_prefill_kernel"], cus=cus), PREFILL) for cus in (256, 8)]
    small = [queue(SMALL, hq, hkv) for hq, hkv in GROUPS] + [queue(([200], [12])), queue(([300] * 40, [1] * 40))]
    want += [(c, EXACT) for c in small] + [(dict(c, out=(1 << 20) + 2), MERGED) for c in small]
    for (c, name), k in zip(want, kernels(tmp, *(c for c, _ in want))):
        assert k[0].startswith(name) and len(k) == (2 if name == MERGED else 1), (c, k)


@pytest.mark.parametrize("sessions,name", [
    (([1999] * 64, [1] * 64), MERGED), (([550, 300], [20, 8]), EXACT), (([2400, 900, 900], [100, 1, 1]), EXACT), (([6000, 900, 900], [30, 1, 1]), MERGED),
    (([2700], [1]), MERGED), (([1100] * 4, [1] * 4), EXACT),
    # more than one workgroup a CU: decodes on contexts past 1800
    (([1799] * 40, [1] * 40), EXACT), (([1819] * 40, [1] * 40), MERGED)])
def test_queue_in_one_kernel_or_two(tmp, sessions, name):
    assert kernels(tmp, queue(sessions, 32, 8))[0][0].startswith(name)


def test_queue_of_few_heads_and_more_than_one_workgroup_a_cu(tmp):
    """Chunks on long contexts go by the merged kernel unless the heads spread over the XCDs."""
    for (hkv, cus, ctx), name in [((8, 256, 3700), EXACT), ((2, 64, 3700), MERGED), ((2, 64, 2100), EXACT), ((2, 256, 2900), EXACT)]:
        c = queue(([ctx] * 12 + [900] * 6, [36] * 12 + [1] * 6), 4 * hkv, hkv, cus=cus)
        assert kernels(tmp, c)[0][0].startswith(name), (hkv, cus, ctx)


@pytest.mark.parametrize("halves,batches", [
    (True, [dict(batch=1, prefix=2000, new=700), dict(batch=1, prefix=2000, new=900, page=32), dict(batch=1, prefix=4000, new=900, d=64), dict(batch=4, new=600, **H82)]),
    (False, [dict(batch=2, prefix=2000, new=700), dict(batch=1, new=480), dict(batch=1, prefix=6000, new=300), dict(batch=8, new=4096)]),
])
def test_two_sets_of_waves_in_a_prefill_workgroup(tmp, halves, batches):
    for b, k in zip(batches, kernels(tmp, *(dict(call="resume", **b) for b in batches))):
        assert len(k) == 1 and k[0].startswith("prefill_halves_kernel") == halves, (b, k)


def test_two_sets_of_waves_in_the_gpu_tests(tmp):
    batches = [dict(call="resume", hq=hq, hkv=1, d=d, page=ps, batch=2, total=sum(new), max_new=max(new), max_ctx=max(p + n for p, n in zip(prefix, new)), cus=8)
               for hq, prefix, new in ACROSS for d, ps in SHAPES]
    for b, k in zip(batches, kernels(tmp, *batches)):
        assert k[0].startswith("prefill_halves_kernel"), (b, k)


# fp32: 1000 tiles of 32 columns to 256 CUs a thousandth; at 32 / 8 heads eight rows are a tile, and a batch of equal sessions of 8 k rows has 8 k tiles a session
@pytest.mark.parametrize("d,prefix,new,most", [
    # 64 channels: one workgroup a CU below 125 tokens, two up to 300, then five thousandths a token more, four at most
    (64, 100, 24, 256), (64, 101, 24, 512), (64, 276, 24, 512), (64, 476, 24, 768), (64, 676, 24, 1024), (64, 3000, 24, 1024),
    # 128: one below 64 tokens, two up to 200, five at most from 800 on
    (128, 39, 24, 256), (128, 40, 24, 512), (128, 176, 24, 512), (128, 376, 24, 768), (128, 776, 24, 1280), (128, 3000, 24, 1280),
])
def test_few_rows_of_fp32(tmp, d, prefix, new, most):
    """The last batch of 24-row chunks, 24 tiles each, that the kernel of few rows takes."""
    batches = [dict(call="resume", dtype="f32", d=d, batch=b, prefix=prefix, new=new) for b in (most // 24, most // 24 + 1)]
    few, tiles = kernels(tmp, *batches)
    assert few[0].startswith(SPLIT) and tiles[0].startswith("prefill_f32_kernel"), (few, tiles)


@pytest.mark.parametrize("shape", [dict(d=128, page=32), dict(dtype="f32", d=64), dict(d=64), dict(d=64, page=32)])
def test_a_grid_at_the_end_of_its_range(tmp, shape):
    """105 KV heads of 20452225 tiles each, 22 short of 2^31 in all: dealt to the XCDs in runs of four they would be 2^31 workgroups,
    one past what a launch may have, and the call is refused; with fewer sessions it is launched."""
    call = dict(call="resume", hq=105, hkv=105, total=0x7fffffff, max_new=640, max_ctx=840, **shape)
    with pytest.raises(AssertionError, match="too many rows"):
        launched([dict(call, batch=4090445)], tmp)
    (k,) = launched([dict(call, batch=4090440)], tmp)
    assert k[0].startswith("prefill_") and int(k[0].rsplit(" ", 1)[1]) <= 0x7fffffff, k
