"""The append of single tokens has two forms that differ in a mark on their stores only, and keeps the compiler from making one of them
with empty asm statements: both forms, as the compiler generates them for gfx950, 16-bit and 32-bit caches."""
import os
import re
import shutil

import pytest

from test_lds_dma_asm import HIPCC, device_asm

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="needs hipcc")


def test_single_tokens_are_stored_both_ways(tmp_path):
    functions = re.split(r"^(?=_ZN\S+:)", device_asm("kv_append.hip", tmp_path), flags=re.M)
    for kernel, element, pieces in (("kv_append_groups_kernelItE", "short", 1), ("kv_append_groups_kernelIjE", "dword", 2)):
        (text,) = [f for f in functions if kernel in f.split(":")[0]]
        stores = [c for c in (line.split(";")[0].strip() for line in text.splitlines()) if c.startswith("global_store")]
        marked = [c.split()[0] for c in stores if c.endswith(" nt")]
        assert sorted(marked) == sorted(["global_store_" + element] + ["global_store_dwordx4"] * pieces), stores
        plain = [c.split()[0] for c in stores if not c.endswith(" nt")]
        # the form without the mark, and that of longer runs: keys, and values a piece or an element at a time
        assert plain.count("global_store_" + element) == 2 and plain.count("global_store_dwordx4") == 3 * pieces, stores
