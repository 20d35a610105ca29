"""The decode step's workgroups count their partials in, and whoever completes a pair reads all of them: a wave's device-scope
stores must have been performed before its workgroup's count is raised.  A workgroup barrier does not wait for them, so this
pins the wait in the code the compiler generates for gfx950; a result that depends on it would be wrong only now and then."""
import os
import shutil

import pytest

from test_lds_dma_asm import HIPCC, device_asm

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="needs hipcc")


def test_partials_are_performed_before_the_count_is_raised(tmp_path):
    ins = [c for c in (line.split(";")[0].strip() for line in device_asm("attn_decode_mfma.hip", tmp_path).splitlines())
           if c and not c.startswith(".") and not c.endswith(":")]
    counts = [i for i, c in enumerate(ins) if c.startswith("global_atomic_add")]
    stores = [i for i, c in enumerate(ins) if c.startswith("global_store") and c.endswith("sc1")]
    assert len(counts) == 1 and stores and max(stores) < counts[0]
    barrier = max(i for i in range(counts[0]) if ins[i] == "s_barrier")
    wait = max(i for i in range(barrier) if ins[i].startswith("s_waitcnt") and "vmcnt(0)" in ins[i])
    assert max(stores) < wait < barrier
    assert not any(c.startswith(("global_store", "s_branch", "s_cbranch")) for c in ins[wait:barrier])
