"""The two ways of the matrix refresh (a workgroup a row where rows are few and short, workgroups by chunk and a merge elsewhere), bit-exact
against the CPU oracle (MI355X only).  The same rows go both ways: 12 slots, or the first six of three sequences of 128."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20104_amd as graft
from gpu_util import dev, host

pytestmark = pytest.mark.gpu
ROW_MAX = 32768              # the longest row of a workgroup of its own


def rows_of(V, rng):
    """Twelve rows: what the threshold, the list of candidates and its ranking can get wrong."""
    x = rng.standard_normal((12, V)).astype(np.float32)
    x[1] = 3.0                                                 # all equal: every element is a candidate
    x[2] = np.sort(x[2])                                       # the largest in one thread or two
    x[3] = -np.sort(-x[3])
    x[4] = np.where(rng.random(V) < 0.5, -0.0, 0.0)            # equal, with either sign
    x[5, rng.integers(0, V, V - min(V, 5))] = -np.inf          # few that are finite
    x[6] = -np.inf
    x[7] = np.round(x[7] * 4) / 4                              # long runs of ties
    x[8, ::7] = 9.0                                            # more ties on top than the list holds
    x[9, -3:] = [7.0, 8.0, 8.0][-V:]                          # behind the last whole group of four
    x[10, :2] = [8.0, 9.0][:V]                               # in front of the first one
    x[11, rng.integers(0, V, 1 + V // 100)] = np.inf
    return x


# lengths around a thread's loads, a wavefront's and the longest row of one workgroup; below k there are fewer elements than places
@pytest.mark.parametrize("V,k", [(1, 1), (3, 3), (16, 16), (17, 16), (67, 8), (1000, 4), (4096, 16), (4099, 9), (8192, 8), (16387, 12),
                                 (ROW_MAX - 1, 8), (ROW_MAX, 16), (ROW_MAX + 1, 16), (50257, 8)])
@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("K", [6, 128])
def test_refresh_both_ways(V, k, shift, K):
    rng = np.random.default_rng(V + k)
    B = 2 if K == 6 else 3
    assert (B * K <= 256) == (K == 6)
    x = rows_of(V, rng)
    n = np.array([6, 6, 0][:B], np.int32)
    tokens = rng.integers(0, V, (B, K)).astype(np.int32)
    tokens[1, 2] = tokens[0, 1]                                # the later one's row stays
    tokens[0, 5] = V
    buf = torch.full((B * K * V + shift + 4,), 100.0, device="cuda")      # what lies around the rows is larger
    lg = buf[shift:shift + B * K * V].view(B, K, V)
    lg[:2, :6] = dev(x.reshape(2, 6, V), "f32")
    M0 = np.full((V, k), -7, np.int32)
    M = dev(M0)
    ids = host(graft.graft_matrix_update(dev(tokens), dev(n), lg, M))
    logits = np.zeros((2, 6, V), np.float32)
    logits[:] = x.reshape(2, 6, V)
    ref = oracle.matrix_update(M0, tokens[:2, :6], n[:2], logits)
    assert (ids[:2, :6] == ref["target_ids"]).all()
    assert (ids[:, 6:] == -1).all() and (ids[2:] == -1).all()
    assert (host(M) == ref["M"]).all()


@pytest.mark.parametrize("B,K", [(2, 128), (257, 1)])
def test_refresh_at_the_line(B, K):
    """256 rows, a workgroup each, and 257: every row, the same tokens again and again."""
    V, k = 1003, 5
    rng = np.random.default_rng(B)
    logits = rng.standard_normal((B, K, V)).astype(np.float32)
    tokens = rng.integers(0, 40, (B, K)).astype(np.int32)
    n = rng.integers(1, K + 1, B).astype(np.int32)
    M0 = np.full((V, k), -7, np.int32)
    M = dev(M0)
    ids = host(graft.graft_matrix_update(dev(tokens), dev(n), dev(logits, "f32"), M))
    ref = oracle.matrix_update(M0, tokens, n, logits)
    assert (ids == ref["target_ids"]).all() and (host(M) == ref["M"]).all()
