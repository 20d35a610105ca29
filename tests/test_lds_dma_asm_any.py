"""The general prefill kernel issues the same direct global-to-LDS loads: the same pins on its generated code."""
import pytest

import test_lds_dma_asm as pins

pytestmark = pins.pytestmark


@pytest.mark.parametrize("src", ["attn_prefill_any.hip"])
def test_m0_belongs_to_the_direct_loads_of_the_general_prefill(src, tmp_path):
    pins.test_m0_belongs_to_the_direct_loads_only(src, tmp_path)
