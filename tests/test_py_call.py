"""The calling module (csrc/py_call.cpp) against the ctypes path it stands in front of: what it does not take raises as before,
and what it takes gives the same bits and the same errors."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_10342_amd import binding as B


def small(device, dtype=torch.bfloat16):
    cache = B.KVCache(8, 16, 2, 128, B.AG_BF16, device, fill=0.0)
    x = lambda *s: torch.zeros(s, dtype=dtype, device=device)
    i = lambda *v: torch.tensor(v, dtype=torch.int32, device=device)
    return cache, x, i


def test_the_module_takes_no_host_tensors_and_ctypes_says_why():
    cache, x, i = small("cpu")
    bt = i(0, 1).view(1, 2)
    args = [cache, x(1, 2, 128), x(1, 2, 128), bt, i(0), i(1), i(0, 1), 1, None]
    assert B._calls().kv_append(*args) is None
    with pytest.raises(ValueError, match="contiguous CUDA"):
        B.ag_kv_append(*args)
    with pytest.raises(TypeError, match="int32"):
        B.ag_attn_prefill(cache, None, None, bt.long(), i(1), i(0, 1), 1, 1, 4, 0.1)
    assert B._calls().kv_append(*args[:-1]) is None                    # too few


def test_without_a_module_that_fits_every_call_goes_through_ctypes(tmp_path, monkeypatch):
    """A missing file, one that is no module, and one built for another torch: a warning, and the calls of before the module."""
    other = tmp_path / "agcall.so"
    other.write_bytes(b"not a module")
    for path, torch_version in [(tmp_path / "nothing.so", torch.__version__), (other, torch.__version__), (B.CALL_PATH, "0.0")]:
        monkeypatch.setattr(B, "_native", None)
        monkeypatch.setattr(B, "CALL_PATH", str(path))
        monkeypatch.setattr(torch, "__version__", torch_version)
        cache, x, i = small("cpu")
        with pytest.warns(RuntimeWarning, match="ctypes"), pytest.raises(ValueError, match="contiguous CUDA"):
            B.ag_kv_append(cache, x(1, 2, 128), x(1, 2, 128), i(0, 1).view(1, 2), i(0), i(1), i(0, 1), 1)
        assert isinstance(B._native, B._NoCalls)
        assert all(getattr(B._calls(), name)(1, 2, 3) is None for name in B._CALLS)


@pytest.mark.gpu
def test_plain_calls_equal_the_ctypes_path_and_others_are_refused_as_there(monkeypatch):
    torch.manual_seed(5)
    cache, x, i = small("cuda")
    n = [20, 1]
    r = lambda *s: torch.randn(s, dtype=torch.bfloat16, device="cuda")
    bt, prefix, new, cu, ctx = i(0, 1, 2, 3).view(2, 2), i(0, 0), i(*n), i(0, 20, 21), i(*n)
    k, v, q = r(21, 2, 128), r(21, 2, 128), r(21, 8, 128)
    ws = torch.zeros(1 << 16, dtype=torch.float32, device="cuda")
    outs = []
    # keywords and positions alike
    side = torch.cuda.Stream()
    for stream, calls in ((None, B._calls()), (torch.cuda.current_stream(), B._calls()), (side, B._calls()), (side.cuda_stream, B._calls()),
                          (None, B._NoCalls()), (side, B._NoCalls())):
        monkeypatch.setattr(B, "_native", calls)
        c2 = B.KVCache(8, 16, 2, 128, B.AG_BF16, "cuda", fill=0.0)
        o = [torch.zeros_like(q) for _ in range(3)] + [torch.zeros_like(q[:2])]
        st, ds, ws2, ctx2 = torch.zeros_like(o[3]), torch.zeros_like(o[3]), torch.zeros(1 << 20, dtype=torch.float32, device="cuda"), i(21, 2)
        torch.cuda.synchronize()                                       # all of it is there, whatever stream the calls run on
        B.ag_kv_append(c2, k, v, bt, prefix_lens=prefix, new_lens=new, cu_new=cu, total_new=21, stream=stream)
        B.ag_attn_prefill(c2, q, o[0], bt, new, cu, 21, 20, 8, 0.09, stream=stream)
        B.ag_attn_resume(c2, q, o[1], bt, prefix, new, cu, 21, 20, 20, 8, 0.09, stream)
        B.ag_attn_merged(c2, q, o[2], bt, prefix, new, cu, 21, 20, 20, 8, 0.09, ws, stream)
        B.ag_attn_decode(c2, q[:2], o[3], bt, ctx, 20, 8, 0.09, ws, stream)
        B.ag_attn_decode_static(c2, q[:2], ds, bt, ctx, 20, 8, 0.09, stream)
        B.ag_decode_step(c2, k[:2], v[:2], q[:2], st, bt, ctx2, 21, 8, 0.09, ws2, stream)
        torch.cuda.synchronize()
        outs.append(o + [st, ds, c2.k_pool, c2.v_pool])
    for same in zip(*outs):
        assert all(torch.equal(a.view(torch.int16), same[0].view(torch.int16)) for a in same) and bool(same[0].any())
    monkeypatch.undo()
    plain = [cache, q[:2], x(2, 8, 128), bt, ctx, 20, 8, 0.09, ws, None]
    call = B._calls().attn_decode
    for stream in (None, torch.cuda.current_stream(), side, torch.cuda.ExternalStream(side.cuda_stream), side.cuda_stream):
        torch.cuda.synchronize()
        assert call(*plain[:9], stream) == B.AG_OK
    torch.cuda.synchronize()
    for at, value in [(1, q[:2, ::2]), (1, q[:2].cpu()), (1, None), (1, torch.nn.Parameter(q[:2].float()).as_subclass(type("T", (torch.Tensor,), {}))),
                      (3, bt.long()), (3, bt[0]), (5, 20.0), (5, np.int32(20)), (5, 1 << 40), (7, 1), (8, None), (9, "s")]:
        args = list(plain)
        args[at] = value
        assert call(*args) is None, at
        if value is None and at == 1:
            with pytest.raises(B.AgError):
                B.ag_attn_decode(*args)
        elif isinstance(value, float):
            with pytest.raises(ctypes.ArgumentError):
                B.ag_attn_decode(*args)
    with pytest.raises(B.AgError) as e:                                # a host-side refusal, through the module
        B.ag_attn_decode(*(plain[:5] + [33] + plain[6:]))
    assert e.value.status == B.AG_ERR_INVALID_ARG and "max_pages" in str(e.value)
