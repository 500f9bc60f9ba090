"""The tests of the MFMA attention kernel with 32-row blocks on its tile of 128 rows (MI355X only): the edges of the tile, splits without a
stage, score and value ranges.  Tolerances as there."""
import pytest

import test_gpu_attn_wide as wide

pytestmark = pytest.mark.gpu

# (B, K, Hq, Hkv, P, tile rows / 64, keys split over workgroups): with and without a last tile that is full
SHAPES = [(8, 33, 64, 4, 700, 2, False), (4, 127, 40, 8, 701, 2, False), (16, 33, 16, 1, 2003, 2, True), (8, 127, 10, 2, 2003, 2, True),
          (2, 128, 40, 8, 2003, 2, True)]


@pytest.fixture(autouse=True)
def plans_say_so(monkeypatch):
    def assert_128(plan, tile, split):
        assert (plan.kernel, plan.row_blocks, plan.splits > 1) == ("tree_attn_wide_128_kernel", tile, split), plan
    monkeypatch.setattr(wide, "assert_wide", assert_128)


shapes = pytest.mark.parametrize("case", SHAPES, ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_tile%d_split%d" % c)


@shapes
@pytest.mark.parametrize("layout", ["head_major", "token_major"])
def test_tiles(case, layout):
    wide.test_tiles(case, layout)


@pytest.mark.parametrize("long_one", [False, True], ids=["all_short", "one_long"])
def test_splits_without_a_stage(long_one):
    wide.test_splits_without_a_stage(SHAPES[3], long_one)


@pytest.mark.parametrize("case", [SHAPES[0], SHAPES[3]], ids=["one_split", "splits"])
@pytest.mark.parametrize("level", wide.LEVELS, ids=lambda x: x.replace(" ", "_"))
def test_score_ranges(case, level):
    wide.test_score_ranges(case, level)


@pytest.mark.parametrize("case", [SHAPES[1], SHAPES[2]], ids=["one_split", "splits"])
def test_tree_slots_far_below_zero(case):
    wide.test_tree_slots_far_below_zero(case)
