"""A workgroup's waves hand tiles to each other through LDS: what one wave overwrites, every wave must have read.  Whether
a barrier stands between the reads and the writes is a property of the generated code, and is checked there, on the CPU:
a missing one gives wrong numbers only when a wave happens to lag."""
import re

import pytest

import test_lds_dma_asm as pins

pytestmark = pins.pytestmark


def steps_of_kernels(text):
    """Per kernel, in program order: 'barrier', 'read' and 'write' (LDS, 16 bytes), 'product'."""
    kinds = (("s_barrier", "barrier"), ("ds_read_b128", "read"), ("ds_write_b128", "write"), ("v_mfma", "product"))
    kernels = {}
    for line in text.splitlines():
        code = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):$", code)
        if m:
            steps = kernels.setdefault(m.group(1), [])
        for op, kind in kinds:
            if code.startswith(op):
                steps.append(kind)
    return {k: v for k, v in kernels.items() if "product" in v}


def test_fp32_prefill_overwrites_the_first_key_tile_behind_a_barrier(tmp_path):
    """The prologue multiplies by the first tile of keys (six products for each k-step of 16 channels); the loop's first
    iteration writes the third tile in its place.  In the loop, one barrier ends an iteration."""
    kernels = steps_of_kernels(pins.device_asm("attn_prefill_f32.hip", tmp_path))
    assert len(kernels) == 2
    for name, steps in kernels.items():
        first = steps.index("product")
        assert "barrier" in steps[:first], name                  # the tile is in LDS before it is read
        write = first + steps[first:].index("write")
        before = steps[first:write]
        assert "barrier" in before, f"{name}: K(0) is overwritten while it may still be read"
        prologue = before[:before.index("barrier")].count("product")
        assert prologue == (24 if "Li64E" in name else 48), (name, prologue)
        assert "barrier" in steps[write:], name
