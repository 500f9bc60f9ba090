"""Which calls take tiles of 128 rows of 32-row blocks: not those whose plan without them has tiles of 64 rows (host code, no GPU needed)."""
import os

import pytest

from gpu_util import attn_plan
from paper_2605_20104_amd import build


@pytest.fixture(autouse=True, scope="module")
def timing_library():
    if not os.path.exists(build.LIB_TIMING):
        build.build_timing()


# us a call with an eighth of the keys that the table has room for, tiles of 64 rows / of 128: 11.3 / 15.3, 11.3 / 15.2, 11.2 / 14.0, 11.2 / 13.8,
# 10.8 / 13.3, 12.1 / 13.8
@pytest.mark.parametrize("B,K,Hkv,G,P", [(2, 61, 1, 4, 37824), (2, 52, 1, 4, 40260), (3, 35, 2, 4, 17019), (2, 68, 2, 2, 29641), (4, 30, 2, 5, 10730),
                                         (1, 80, 2, 2, 64575)])
def test_tiles_of_64_rows_stay(B, K, Hkv, G, P):
    plan = attn_plan(B, K, G * Hkv, Hkv, 128, -(-(P + K) // 16), "bf16")
    assert (plan.kernel, plan.row_blocks) == ("tree_attn_mfma_kernel", 1), plan


# in place of tiles of 128 rows of 16-row blocks, of 192 and of 256 rows: 13.3 / 12.9, 18.9 / 14.3 and 19.3 / 15.6 us with an eighth of the keys
@pytest.mark.parametrize("B,K,Hkv,G,P", [(12, 112, 4, 4, 1221), (5, 86, 2, 4, 8397), (3, 58, 8, 4, 8276)])
def test_other_tiles_give_way(B, K, Hkv, G, P):
    plan = attn_plan(B, K, G * Hkv, Hkv, 128, -(-(P + K) // 16), "bf16")
    assert (plan.kernel, plan.row_blocks) == ("tree_attn_wide_128_kernel", 2), plan
