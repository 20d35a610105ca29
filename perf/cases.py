"""The performance cases of the library: the work a serving engine has it do, through its public entry points.

A case is a dict of plain values.  `kind` says which calls a pass makes:
  step     one decode step in one launch (ag_decode_step: append of the step's token + attention)
  decode   one decode step as two calls (ag_kv_append, ag_attn_decode): every cache the library supports
  cold     a cold prefill (ag_kv_append, ag_attn_prefill): whole prompts
  resume   a resume prefill (ag_kv_append, ag_attn_resume): chunks appended to cached prefixes
  queue    the scheduler's decode queue (ag_kv_append, ag_attn_merged): decodes and short chunks in one batch
  session  a whole small session: cold prefill, resume prefill, then decode steps one after the other
Geometry: `hq` / `hkv` query and KV heads, `d` channels, `page` tokens a page, `dtype` of cache and activations.
Sizes: `batch` sessions with `p_lo`..`p_hi` cached tokens and `n_lo`..`n_hi` new ones (for step and decode the
new token is the step's own), drawn from `lens`; `decodes` sessions of a queue bring one row on c_lo..c_hi.

Values are N(0, 1): logits of standard deviation about 1, as normalised queries and keys have.  Pages that a
session does not use, and slots behind its last token, hold stale finite values, as a pool in use does.
"""
import math

import numpy as np
import torch

from paper_2603_10342_amd import binding as B

DEV = "cuda"


def _case(name, kind, dtype="bf16", hq=32, hkv=8, d=128, page=16, batch=1, p=(0, 0), n=(1, 1), lens=1, **more):
    c = {"kind": kind, "dtype": dtype, "hq": hq, "hkv": hkv, "d": d, "page": page, "batch": batch, "p_lo": p[0],
         "p_hi": p[1], "n_lo": n[0], "n_hi": n[1], "lens": lens}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one agent decoding alone: the shortest call, all latency
        _case("step_1", "step", batch=1, p=(999, 999)),
        # the decode-only benchmark workload: 64 sessions, contexts 1024..4096
        _case("decode_64", "decode", batch=64, p=(1023, 4095), lens=2),
        # the decode side of the mixed workload: 64 sessions, contexts 1024..8192, one launch
        _case("step_64", "step", batch=64, p=(1023, 8191), lens=5),
        # the cold-prefill benchmark workload: 8 system prompts of 4096 tokens
        _case("cold_8x4096", "cold", batch=8, n=(4096, 4096), lens=3),
        # the resume-prefill benchmark workload: 32 chunks of 128..1024 rows on 2048..8192 cached tokens
        _case("resume_32", "resume", batch=32, p=(2048, 8192), n=(128, 1024), lens=4),
        # one agent's tool output comes back: one ragged chunk on a long prefix
        _case("resume_1", "resume", batch=1, p=(6007, 6007), n=(211, 211)),
        # the scheduler's decode queue: 64 decodes and 8 tool outputs of 16..64 rows
        _case("queue_72", "queue", batch=8, p=(2048, 8192), n=(16, 64), lens=6, decodes=64, c_lo=1024, c_hi=4096),
        # the small end-to-end configuration: fp32, 4/2 heads, head_dim 64, cold 256, resume 32, 16 decode steps
        _case("session_f32", "session", dtype="f32", hq=4, hkv=2, d=64, batch=2, n=(256, 256), resume=32, steps=16),
        # fp32 caches at the benchmark's head counts: decode and prompt
        _case("decode_f32", "decode", dtype="f32", batch=16, p=(1023, 4095), lens=7),
        _case("cold_f32", "cold", dtype="f32", batch=4, n=(300, 1500), lens=8),
        # other geometries: half-width heads on larger pages, decode and tool outputs
        _case("decode_d64_p32", "decode", d=64, page=32, batch=48, p=(700, 5000), lens=9),
        _case("resume_d64_p64", "resume", d=64, page=64, batch=8, p=(500, 4000), n=(40, 500), lens=10),
    ]


# ---- sizes ----

def _pairs(p, n):
    return int((n * p + n * (n + 1) // 2).sum())


def lengths(case):
    """(cached, new) tokens of every session, as int64 arrays."""
    rng = np.random.default_rng(case["lens"])
    b = case["batch"]
    p = rng.integers(case["p_lo"], case["p_hi"] + 1, size=b)
    n = rng.integers(case["n_lo"], case["n_hi"] + 1, size=b)
    if case["kind"] == "queue":
        ctx = rng.integers(case["c_lo"], case["c_hi"] + 1, size=case["decodes"])
        p = np.concatenate([ctx - 1, p])
        n = np.concatenate([np.ones(len(ctx), p.dtype), n])
    return p.astype(np.int64), n.astype(np.int64)


def phases(case):
    """The (kind, cached, new) of every append + attention pair of a pass."""
    p, n = lengths(case)
    if case["kind"] != "session":
        return [(case["kind"], p, n)]
    out = [("cold", p, n), ("resume", n, np.full_like(n, case["resume"]))]
    at = n + case["resume"]
    return out + [("decode", at + i, np.ones_like(n)) for i in range(case["steps"])]


def work(case):
    el = 4 if case["dtype"] == "f32" else 2
    nbytes = flops = 0
    for _, p, n in phases(case):
        token = 2 * case["hkv"] * case["d"] * el                          # one token's keys and values
        nbytes += int(p.sum()) * token + 2 * int(n.sum()) * token         # cached ones read; new ones read and written
        nbytes += 2 * int(n.sum()) * case["hq"] * case["d"] * el          # queries and outputs
        nbytes += 4 * int(((p + n + case["page"] - 1) // case["page"]).sum())
        flops += 4 * case["d"] * case["hq"] * _pairs(p, n)
    return {"bytes": nbytes, "flops": flops}


GENERAL_FLOPS = 6e10         # what a drawn prefill of the geometries beside the benchmark's may cost
MAIN_FLOPS = 1.5e12          # ... and one of the benchmark's


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "decode", "decode", "cold", "cold", "resume", "resume", "queue"])
    main = kind == "step" or rng.random() < 0.5
    if main:
        geo = dict(dtype="bf16", d=128, page=16)
    else:
        geo = dict(rng.choice([dict(dtype="bf16", d=64, page=16), dict(dtype="bf16", d=64, page=32),
                               dict(dtype="bf16", d=64, page=64), dict(dtype="bf16", d=128, page=32),
                               dict(dtype="bf16", d=128, page=64), dict(dtype="bf16", d=256, page=16),
                               dict(dtype="f32", d=64, page=16), dict(dtype="f32", d=128, page=16),
                               dict(dtype="f32", d=64, page=32)]))
    hq, hkv = rng.choice([(32, 8), (32, 8), (32, 8), (8, 2), (16, 2), (4, 4), (6, 2), (16, 1)])
    lens = rng.randrange(1, 1 << 30)
    lo = log(64, 2048)
    if kind in ("step", "decode"):
        hi = log(lo, 8192 if main else 4096)
        return _case(None, kind, hq=hq, hkv=hkv, batch=log(1, 64 if main else 32), p=(lo, hi), lens=lens, **geo)
    if kind == "queue":
        hi = log(lo, 8192 if main else 4096)
        n_lo = log(2, 32)
        c = _case(None, kind, hq=hq, hkv=hkv, batch=log(1, 8), p=(lo, hi), n=(n_lo, log(n_lo, 128)), lens=lens,
                  decodes=log(1, 64 if main else 16), c_lo=log(64, 1024), c_hi=log(1024, 4096), **geo)
    elif kind == "cold":
        n_lo = log(16, 2048 if main else 800)
        c = _case(None, kind, hq=hq, hkv=hkv, batch=log(1, 16), n=(n_lo, log(n_lo, 4096 if main else 1500)), lens=lens, **geo)
    else:
        hi = log(lo, 8192 if main else 4096)
        n_lo = log(4, 256)
        c = _case(None, kind, hq=hq, hkv=hkv, batch=log(1, 32), p=(lo, hi), n=(n_lo, log(n_lo, 1024 if main else 512)), lens=lens, **geo)
    while c["batch"] > 1 and work(c)["flops"] > (MAIN_FLOPS if main else GENERAL_FLOPS):
        c["batch"] //= 2
    return c


# ---- a pass ----

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _inputs(case, seed):
    """Everything that is drawn: pools, block tables, and queries, keys and values of every phase."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    dt, hq, hkv, d, ps = _dtype(case), case["hq"], case["hkv"], case["d"], case["page"]

    def values(*shape):
        return torch.randn(shape, dtype=dt, device=DEV, generator=gen)

    ph = phases(case)
    need = (ph[-1][1] + ph[-1][2] + ps - 1) // ps
    pages = int(need.sum()) + 16
    rng = np.random.default_rng(int(seed))
    perm = rng.permutation(pages)
    bt = np.zeros((len(need), int(need.max())), np.int32)                  # unused entries name a valid page, as stale rows do
    at = 0
    for s, k in enumerate(need):
        bt[s, :k] = perm[at:at + k]
        at += k
    cache = B.KVCache(pages, ps, hkv, d, B.AG_F32 if case["dtype"] == "f32" else B.AG_BF16, DEV)
    cache.k_pool = values(*cache.k_pool.shape)
    cache.v_pool = values(*cache.v_pool.shape)
    batches = []
    for kind, p, n in ph:
        t = int(n.sum())
        batches.append({"kind": kind, "p": p, "n": n, "q": values(t, hq, d), "k": values(t, hkv, d), "v": values(t, hkv, d)})
    return cache, bt, batches


def prepare(case, seed):
    cache, bt, batches = _inputs(case, seed)
    hq, d = case["hq"], case["d"]
    for b in batches:
        p, n = b.pop("p"), b.pop("n")
        b["total"], b["max_new"], b["max_ctx"] = int(n.sum()), int(n.max()), int((p + n).max())
        b["prefix"], b["new"], b["ctx"] = _i32(p), _i32(n), _i32(p + n)
        b["cu"] = _i32(np.concatenate([[0], np.cumsum(n)]))
        b["out"] = torch.empty_like(b["q"])
        nbytes = 0
        if b["kind"] == "decode":
            nbytes = B.ag_attn_decode_workspace_bytes(len(n), hq, d, b["max_ctx"])
        elif b["kind"] == "step":
            nbytes = B.ag_decode_step_workspace_bytes(len(n), hq, d, b["max_ctx"])
        elif b["kind"] == "queue":
            nbytes = B.ag_attn_merged_workspace_bytes(b["total"], hq, b["max_ctx"])
        b["ws"] = torch.zeros((nbytes + 15) // 16 * 4 + 4, dtype=torch.float32, device=DEV)
    return {"cache": cache, "bt": _i32(bt), "batches": batches, "hq": hq, "scale": 1.0 / math.sqrt(d)}


def run(state):
    cache, bt, hq, scale = state["cache"], state["bt"], state["hq"], state["scale"]
    outs = []
    for b in state["batches"]:
        kind = b["kind"]
        if kind == "step":
            B.ag_decode_step(cache, b["k"], b["v"], b["q"], b["out"], bt, b["ctx"], b["max_ctx"], hq, scale, b["ws"])
        else:
            B.ag_kv_append(cache, b["k"], b["v"], bt, b["prefix"], b["new"], b["cu"], b["total"])
        if kind == "decode":
            B.ag_attn_decode(cache, b["q"], b["out"], bt, b["ctx"], b["max_ctx"], hq, scale, b["ws"])
        elif kind == "cold":
            B.ag_attn_prefill(cache, b["q"], b["out"], bt, b["new"], b["cu"], b["total"], b["max_new"], hq, scale)
        elif kind == "resume":
            B.ag_attn_resume(cache, b["q"], b["out"], bt, b["prefix"], b["new"], b["cu"], b["total"], b["max_new"],
                             b["max_ctx"], hq, scale)
        elif kind == "queue":
            B.ag_attn_merged(cache, b["q"], b["out"], bt, b["prefix"], b["new"], b["cu"], b["total"], b["max_new"],
                             b["max_ctx"], hq, scale, b["ws"])
        outs.append(b["out"])
    return {"out": outs, "k_pool": cache.k_pool, "v_pool": cache.v_pool}


# ---- the same in 64 bits ----

def _v_index(slots):
    """Chunk of eight and position inside it at which a value page stores a slot."""
    return ((slots >> 4) << 1) | ((slots >> 2) & 1), (slots & 3) | (((slots >> 3) & 1) << 2)


def exact(case, seed):
    cache, bt, batches = _inputs(case, seed)
    kp, vp = cache.k_pool, cache.v_pool
    hq, hkv, d, ps = case["hq"], case["hkv"], case["d"], case["page"]
    g, scale = hq // hkv, 1.0 / math.sqrt(d)
    chunk, pos = _v_index(torch.arange(ps, device=DEV))
    outs = []
    for b in batches:
        out = torch.empty(b["q"].shape, dtype=torch.float64, device=DEV)
        row = 0
        for s, (p, n) in enumerate(zip(b["p"].tolist(), b["n"].tolist())):
            table = torch.from_numpy(bt[s].astype(np.int64)).to(DEV)
            j = torch.arange(p, p + n, device=DEV)
            pages, slots = table[j // ps], j % ps
            kp[pages, :, :, slots, :] = b["k"][row:row + n].view(n, hkv, d // 8, 8)
            c, e = _v_index(slots)
            vp[pages, :, c, :, e] = b["v"][row:row + n]
            used = table[:(p + n + ps - 1) // ps]
            k = kp[used].permute(1, 0, 3, 2, 4).reshape(hkv, -1, d)[:, :p + n].double()
            v = vp[used][:, :, chunk, :, pos].permute(2, 1, 0, 3).reshape(hkv, -1, d)[:, :p + n].double()
            q = b["q"][row:row + n].double().view(n, hkv, g, d)
            hidden = torch.arange(p + n, device=DEV)[None, :] > j[:, None]
            for h in range(hkv):
                x = (q[:, h].reshape(n * g, d) @ k[h].t().contiguous()) * scale
                x = x.view(n, g, p + n).masked_fill_(hidden[:, None, :], -math.inf)
                out[row:row + n, h * g:(h + 1) * g] = (torch.softmax(x, -1).view(n * g, p + n) @ v[h]).view(n, g, d)
            row += n
        outs.append(out)
    return {"out": outs, "k_pool": None, "v_pool": None}


def tolerance(case):
    # About four times what the paths show against exact().  bf16: 1.6e-3 to 2.4e-3 in norm (weights and outputs rounded
    # to 8 bits), 4.5e-2 at most in one value (early rows of a cold prompt).  fp32: 4e-7 to 1e-6 in norm and 9e-6 in one
    # value (sums of up to 4096 keys).
    return {"rel": 4e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.18}
