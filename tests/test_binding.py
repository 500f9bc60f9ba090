"""The native marshalling of the Python binding (no GPU): arguments that do not fit are Python errors,
argument errors of the library are GraftError, and nothing is launched in either case."""
import pytest
import torch

import paper_2605_20104_amd as graft


def _mask(parent=None, n_leaf_max=4, depth_cap=200, out=None):
    one = torch.ones(2, dtype=torch.int32)
    parent = torch.zeros((2, 8), dtype=torch.int32) if parent is None else parent
    return graft.graft_build_tree_mask(parent, one, one, n_leaf_max, depth_cap, out=out, stream=0)


@pytest.mark.parametrize("kwargs,error", [
    (dict(parent=torch.zeros((8, 2), dtype=torch.int32).t()), AssertionError),       # not dense row-major
    (dict(parent=torch.zeros(8, dtype=torch.int32)), ValueError),                    # not [B, K]
    (dict(parent=3), TypeError),
    (dict(out={}), KeyError),                                                        # an output is missing
    (dict(n_leaf_max="4"), TypeError),
])
def test_arguments_that_do_not_fit(kwargs, error):
    with pytest.raises(error):
        _mask(**kwargs)


def test_library_errors_carry_their_code():
    with pytest.raises(graft.GraftError) as e:
        _mask(depth_cap=200)
    assert e.value.code == graft.GRAFT_ERR_SHAPE and "graft_build_tree_mask" in str(e.value)
    q = torch.zeros((1, 4, 8, 96), dtype=torch.bfloat16)
    with pytest.raises(graft.GraftError) as e:
        graft.graft_tree_attn(q, q, q, {"page": 1536, "token": 96, "head": 96}, torch.zeros((1, 2), dtype=torch.int32), *(
            [torch.zeros(1, dtype=torch.int32)] * 2), torch.zeros((1, 4, 2), dtype=torch.int64), 2, 0.1, stream=0)
    assert e.value.code == graft.GRAFT_ERR_SHAPE
    with pytest.raises(AssertionError):                                               # mixed storage types
        graft.graft_tree_attn(q, q.float(), q, {"page": 1, "token": 1, "head": 1}, torch.zeros((1, 2), dtype=torch.int32),
                              None, None, None, 2, 0.1, stream=0)
