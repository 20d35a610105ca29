"""bf16 / 128 / page 16 decode in shares: what a step's arithmetic promises, read from the workspace that the split kernel leaves
behind."""
import numpy as np
import pytest
import torch

from gpu_helpers import DevBatch, gpu_append, i32, make_cache
from helpers import make_batch
from paper_2603_10342_amd import binding as B
from paper_2603_10342_amd import inputs as I

pytestmark = pytest.mark.gpu

STEP, MIN_STEPS = 32, 8


def split_workspace(batch, g, max_ctx):
    """The workspace of ag_attn_decode, and where its parts lie: [share, steps before each session], O, (m, l)."""
    ws = torch.zeros(B.ag_attn_decode_workspace_bytes(batch, g.num_q_heads, g.head_dim, max_ctx) // 4, dtype=torch.float32, device="cuda")
    pieces = ((max_ctx + STEP - 1) // STEP - 1) // MIN_STEPS + 2
    header = (batch + 4) & ~3
    ml = header + batch * g.num_q_heads * pieces * g.head_dim
    return ws, pieces, ml


def test_equal_scores_have_equal_weights():
    """Every key the same and a score that rounding changes: each weight is exactly 1, and a part's sum the number of its tokens."""
    g = I.Geometry(16, 1, 128, 16, 100, I.BF16)
    ctx = 1300
    fill = make_batch(g, [0], [ctx], seed=81, sigma_qk=2.5, sigma_v=1.0)
    fill.k_new[:] = fill.k_new[:1]
    cache = make_cache(g)
    df = DevBatch(fill)
    gpu_append(cache, df)
    q = df.q[:1].contiguous()
    ws, pieces, ml = split_workspace(1, g, ctx)
    B.ag_attn_decode(cache, q, torch.empty_like(q), df.bt, i32([ctx]), ctx, g.num_q_heads, g.scale, ws)
    torch.cuda.synchronize()
    share = int(ws[:1].view(torch.int32)[0])
    m, l = ws[ml:ml + 16 * pieces * 2].view(16, pieces, 2).cpu().numpy().transpose(2, 0, 1)
    used = -(-ctx // (share * STEP))
    assert share == MIN_STEPS and np.abs(m[:, 0]).max() > 16           # half a unit in the last place there is 1e-6, ten times that of a weight
    assert np.array_equal(l[:, :used], np.broadcast_to(np.minimum(share * STEP, ctx - np.arange(used) * share * STEP), (16, used)).astype(np.float32))
