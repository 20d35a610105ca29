"""Which kernels a call launches, seen without a GPU: libagattn.so is loaded in a process of its own behind a HIP runtime that
only logs (tests/hostbuild/launch_log.cpp), and called through ctypes with addresses that nothing reads.

    launched([dict(call="resume", d=128, batch=2, prefix=100, new=50), ...]) -> [["kernel<..> workgroups", ...], ...]
"""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_10342_amd", "libagattn.so")
SHAPE = dict(dtype="bf16", d=128, page=16, hq=32, hkv=8, cus=256, out=1 << 20)


def launched(calls, tmp):
    """calls: dicts with call = cold | resume | merged | decode | step, the shape (SHAPE where left out), and either batch,
    prefix and new (equal sessions) or total, batch, max_new and max_ctx.  cus: those of the stream."""
    so = os.path.join(str(tmp), "launch_log.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", os.path.join(ROOT, "tests", "hostbuild", "launch_log.cpp"), "-o", so],
                       check=True, capture_output=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so, LIB], input=json.dumps([{**SHAPE, **c} for c in calls]),
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout)


def _main(log_so, lib_so):
    import ctypes as C
    log = C.CDLL(log_so, mode=C.RTLD_GLOBAL)
    log.launch_log_take.restype = C.c_char_p
    lib = C.CDLL(lib_so)
    lib.ag_last_error.restype = C.c_char_p
    for f in ("ag_attn_decode_workspace_bytes", "ag_decode_step_workspace_bytes", "ag_attn_merged_workspace_bytes"):
        getattr(lib, f).restype = C.c_size_t

    class Cache(C.Structure):
        _fields_ = [("k_pool", C.c_void_p), ("v_pool", C.c_void_p)] + [(n, C.c_int32) for n in ("num_pages", "page_size", "num_kv_heads", "head_dim", "dtype")]

    p, f = C.c_void_p, C.c_float
    any_ = 1 << 20                                                     # an aligned address that nothing reads
    results = []
    for c in json.loads(sys.stdin.read()):
        batch = c["batch"]
        new = c.get("new", 1)
        total = c.get("total", batch * new)
        max_new = c.get("max_new", new)
        max_ctx = c.get("max_ctx", c.get("prefix", 0) + new)
        cache = Cache(any_, any_, 1 << 20, c["page"], c["hkv"], c["d"], 1 if c["dtype"] == "bf16" else 0)
        pages = -(-max_ctx // c["page"])
        stream = p(c["cus"] if c["cus"] != 256 else 0)
        q, out, bt, lens, scale = p(any_), p(c["out"]), p(any_), p(any_), f(0.1)
        log.launch_log_take()
        if c["call"] == "cold":
            st = lib.ag_attn_prefill(C.byref(cache), q, out, bt, pages, lens, lens, batch, total, max_new, c["hq"], scale, stream)
        elif c["call"] == "resume":
            st = lib.ag_attn_resume(C.byref(cache), q, out, bt, pages, lens, lens, lens, batch, total, max_new, max_ctx, c["hq"], scale, stream)
        elif c["call"] == "merged":
            n = lib.ag_attn_merged_workspace_bytes(total, c["hq"], max_ctx)
            st = lib.ag_attn_merged(C.byref(cache), q, out, bt, pages, lens, lens, lens, batch, total, max_new, max_ctx, c["hq"], scale, p(any_),
                                    C.c_size_t(n), stream)
        elif c["call"] == "decode":
            n = lib.ag_attn_decode_workspace_bytes(batch, c["hq"], c["d"], max_ctx)
            st = lib.ag_attn_decode(C.byref(cache), q, out, bt, pages, lens, batch, max_ctx, c["hq"], scale, p(any_), C.c_size_t(n), stream)
        else:
            n = lib.ag_decode_step_workspace_bytes(batch, c["hq"], c["d"], max_ctx)
            st = lib.ag_decode_step(C.byref(cache), p(any_), p(any_), q, out, bt, pages, lens, batch, max_ctx, c["hq"], scale, p(any_), C.c_size_t(n), stream)
        assert st == 0, (c, st, lib.ag_last_error())
        results.append(log.launch_log_take().decode().split("\n")[:-1])
    print(json.dumps(results))


if __name__ == "__main__":
    _main(*sys.argv[1:])
