"""Which attention path a shape takes, where a limit decides it (host code, no GPU needed)."""
import os

import pytest

from gpu_util import attn_plan
from paper_2605_20104_amd import build


@pytest.mark.parametrize("K,Hq,Hkv,forced", [(128, 131072, 16384, True), (127, 131072, 16384, False), (128, 131056, 16382, False), (1, 1048560, 65535, False)])
def test_queries_past_what_a_buffer_descriptor_holds_take_the_direct_path(K, Hq, Hkv, forced):
    """The MFMA path reads a sequence's queries through a buffer descriptor, which ends before 4 GB: K Hq rows of 256 bytes."""
    if not os.path.exists(build.LIB_TIMING):
        pytest.skip("libgraft_timing.so is not built")
    assert (K * Hq * 256 >= 1 << 32) == forced
    plan = attn_plan(1, K, Hq, Hkv, 128, 4096, "bf16")
    if forced:
        assert plan.path == "direct", plan
    elif K > 100:
        assert plan.path == "mfma", plan
