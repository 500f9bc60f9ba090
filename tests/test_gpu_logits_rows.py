"""The scans of logits rows (acceptance, matrix refresh) at every cut of a row into 16-byte groups: lengths and
addresses that are no multiple of it, rows shorter than the workgroups that share them, chunks longer than
the registers, runs of equal values, -inf and NaN.  Whole numbers: exact (MI355X only)."""
import numpy as np
import pytest
import torch

import paper_2605_20104_amd as graft

pytestmark = pytest.mark.gpu

# 196608 = 16 chunks of 12 16-byte loads by 256 threads
LENGTHS = [1, 2, 3, 4, 5, 7, 16, 63, 64, 67, 1000, 4099, 16385, 50257, 151936, 196608, 196609, 196615, 262147]


def best(row, k):
    """Ids of the k largest, the smaller id first among equals; NaN is never chosen, -1 where nothing is left."""
    order = np.lexsort((np.arange(len(row)), -row))
    return (order[~np.isnan(row[order])][:k].tolist() + [-1] * k)[:k]


@pytest.mark.parametrize("V", LENGTHS)
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_rows_of_any_length_and_address(V, shift):
    rng = np.random.default_rng(V + shift)
    B, K, k = 2, 5, min(8, V)
    logits = rng.standard_normal((B, K, V)).astype(np.float32)
    logits[0, 1, -1] = logits[0, 1, 0] = 9.0                               # first and last element, equal
    logits[0, 2] = np.round(logits[0, 2])                                  # long runs of equal values
    logits[0, 3, : V - 1] = -np.inf
    logits[1, 0, V // 2:] = 7.0
    logits[1, 1, ::2] = np.nan
    logits[1, 1, V - 1] = 20.0
    logits[1, 3, : max(0, V - 2)] = logits[1, 3, : max(0, V - 2)].clip(max=3.0)
    logits[1, 3, -1] = 11.0                                                # the tail alone
    buf = torch.full((logits.size + shift + 4,), 100.0, device="cuda")     # what lies around the rows is larger
    lg = buf[shift:shift + logits.size].view(B, K, V)
    lg.copy_(torch.from_numpy(logits))
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    parent = np.tile(np.arange(-1, K - 1), (B, 1))
    tokens = np.stack([(np.arange(K) + 5 * b) % V for b in range(B)])
    n = up([K, K - 1])
    want = np.array([[best(logits[b, i], 1)[0] if i < K - b else -1 for i in range(K)] for b in range(B)])

    acc = graft.graft_accept(up(parent), up(tokens), n, 8, logits=lg)
    assert (acc["target_ids"].cpu().numpy() == want).all()

    M = torch.full((V, k), -7, dtype=torch.int32, device="cuda")
    ids = graft.graft_matrix_update(up(tokens), n, lg, M)
    assert (ids.cpu().numpy() == want).all()
    rows = {}
    for b in range(B):
        for i in range(K - b):
            rows[int(tokens[b, i])] = best(logits[b, i], k)
    # (a token met twice: the later node's row is there, and rows[] was filled in the same order)
    want_M = np.full((V, k), -7, np.int32)
    for t, r in rows.items():
        want_M[t] = r                                                      # ids, then -1 where no candidate is left
    assert (M.cpu().numpy() == want_M).all()


@pytest.mark.parametrize("V", [1, 2, 3, 6, 1000, 8191, 8192, 8195, 8196, 8199, 16389])
@pytest.mark.parametrize("shift,rows", [(0, 2048), (1, 2048), (3, 2048), (3, 1024), (2, 192)])
def test_rows_cut_by_their_number(V, shift, rows):
    """Many rows go to as few workgroups as take 8192 elements each (both edges in one where it is alone), fewer
    rows to as many as fill the chip."""
    rng = np.random.default_rng(V + shift)
    K, k, used = 64, min(8, V), 3
    B = rows // K
    logits = torch.randn(rows * V, generator=torch.Generator(device="cuda").manual_seed(V), device="cuda")
    buf = torch.full((rows * V + shift + 4,), 100.0, device="cuda")
    lg = buf[shift:shift + rows * V].view(B, K, V)
    lg.copy_(logits.view(B, K, V))
    lg[0, 0, -1] = lg[0, 0, 0] = 9.0                                       # first and last element, equal
    lg[0, 1, -1] = 11.0
    lg[0, 2] = lg[0, 2].round()                                            # long runs of equal values
    lg[1, 0, : V - 1] = -np.inf
    lg[1, 1, ::2] = np.nan
    lg[1, 1, V - 1] = 20.0
    host = lg[:, :used].cpu().numpy()
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    parent = np.tile(np.arange(-1, K - 1), (B, 1))
    tokens = rng.integers(0, V, (B, K))
    n = up([used] * B)
    want = np.full((B, K), -1)
    rows_of = {}
    for b in range(B):
        for i in range(used):
            order = best(host[b, i], k)
            want[b, i] = order[0]
            rows_of[int(tokens[b, i])] = order                             # the later node's row stays
    acc = graft.graft_accept(up(parent), up(tokens), n, 8, logits=lg)
    assert (acc["target_ids"].cpu().numpy() == want).all()
    M = torch.full((V, k), -7, dtype=torch.int32, device="cuda")
    ids = graft.graft_matrix_update(up(tokens), n, lg, M)
    assert (ids.cpu().numpy() == want).all()
    want_M = np.full((V, k), -7, np.int32)
    for t, r in rows_of.items():
        want_M[t] = r
    assert (M.cpu().numpy() == want_M).all()
