"""Which fp32 calls take the kernel on the 16-bit matrix cores: none that are slower so (host code, no GPU needed)."""
import os

import pytest

from gpu_util import attn_plan
from paper_2605_20104_amd import build


@pytest.fixture(autouse=True, scope="module")
def timing_library():
    if not os.path.exists(build.LIB_TIMING):
        build.build_timing()


def kernel(B, K, Hkv, G, P, D):
    return attn_plan(B, K, G * Hkv, Hkv, D, -(-(P + K) // 16), "f32").kernel


# us a call with fp32 products / on the 16-bit matrix cores, with a full table and with half of its keys: 32.7 / 36.4 and 18.0 / 21.1, 32.5 / 35.8 and
# 26.8 / 33.4, 65.1 / 67.6 and 41.6 / 49.8, 65.4 / 66.7 and 41.9 / 49.7, 62.1 / 65.5 and 37.8 / 40.9, 63.5 / 60.6 and 41.1 / 44.1
@pytest.mark.parametrize("B,K,Hkv,G,P,D", [(7, 66, 4, 2, 2807, 64), (3, 128, 8, 12, 91, 64), (9, 58, 8, 13, 374, 64), (10, 82, 8, 8, 335, 64),
                                           (6, 110, 4, 3, 1422, 128), (7, 71, 4, 15, 332, 128)])
def test_slower_ones_stay(B, K, Hkv, G, P, D):
    assert kernel(B, K, Hkv, G, P, D) == "tree_attn_direct_kernel"


# 22.6 / 17.3; 96.8 / 65.5; 38.6 / 29.8 and 24.7 / 24.8; 155.2 / 117.2 and 99.6 / 84.9; 59.5 / 54.3 and 33.0 / 32.4
@pytest.mark.parametrize("B,K,Hkv,G,P,D", [(1, 40, 8, 4, 2048, 128), (1, 64, 8, 5, 8192, 128), (9, 66, 2, 16, 389, 64), (8, 121, 4, 14, 430, 128),
                                           (7, 42, 4, 1, 15831, 64)])
def test_faster_ones_change(B, K, Hkv, G, P, D):
    assert kernel(B, K, Hkv, G, P, D) == "tree_attn_parts_kernel"
