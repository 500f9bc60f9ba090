"""Which attention path a shape takes, where a limit decides it (host code, no GPU needed)."""
import os
import random

import pytest

from gpu_util import attn_plan
from paper_2605_20104_amd import build


@pytest.fixture(autouse=True, scope="module")
def timing_library():
    if not os.path.exists(build.LIB_TIMING):
        build.build_timing()


@pytest.mark.parametrize("K,Hq,Hkv,forced", [(128, 131072, 16384, True), (127, 131072, 16384, False), (128, 131056, 16382, False)])
def test_queries_past_what_a_buffer_descriptor_holds_take_the_direct_path(K, Hq, Hkv, forced):
    """The MFMA path reads a sequence's queries through a buffer descriptor, which ends before 4 GB: K Hq rows of 256 bytes."""
    assert (K * Hq * 256 >= 1 << 32) == forced
    plan = attn_plan(1, K, Hq, Hkv, 128, 4096, "bf16")
    assert plan.path == ("direct" if forced else "mfma"), plan


def test_32_row_blocks_have_enough_stages_a_split():
    """Tiles of 192 rows from 11 stages on, of 384 rows too where the keys are split: the fixed part and the partial rows of
    shorter splits cost more than the loop gains."""
    rng = random.Random(8)
    seen = set()
    for _ in range(4000):
        B, Hkv, G, K, pages = rng.randint(1, 16), rng.choice([1, 2, 4, 8]), rng.randint(1, 16), rng.randint(8, 128), int(2 ** rng.uniform(2, 12))
        plan = attn_plan(B, K, G * Hkv, Hkv, 128, pages, "bf16")
        if plan.kernel != "tree_attn_wide_kernel":
            continue
        stages = -(-(-(-pages // 4)) // plan.splits)
        seen.add((plan.row_blocks, plan.splits > 1, stages >= 11))
        assert plan.row_blocks in (3, 4, 6), plan
        if plan.row_blocks == 3 or (plan.row_blocks == 6 and plan.splits > 1):
            assert stages >= 11, (plan, pages)
    assert {(3, False, True), (3, True, True), (4, True, False), (6, False, False), (6, True, True)} <= seen, seen
    # (5 splits of 5 stages in 3 tiles of 384 rows before: 33.7 us, 31.1 with 16-row blocks, 30.0 now)
    assert attn_plan(4, 96, 48, 4, 128, 100, "bf16")[1:4] == (4, 5, 3)
