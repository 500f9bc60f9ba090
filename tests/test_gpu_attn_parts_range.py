"""fp32 attention on the matrix cores where operands of very different size meet in a tile, against 64-bit arithmetic (MI355X only).

Bound of a result in dim d of a row, every part of it for that row alone.  A score is off by at most 29 * 2^-24 of sum |q k| (operands
of 23 bits, 24 partial sums) and, where operands lose bits below fp16's, by what the kernel lets pass: 2^-22 of the largest score in
units of ln 2, at least 2^-22, as a root mean square; four times that here.  A weight p is off by that part of itself, and the
weights' sum by the weighted mean of it.  Probabilities and values keep their 24 bits, of their products up to 2^-22 is left out,
and a sum is rounded twelve times a tile and once a wavefront, split and merge: (5 + 12 tiles + 48) 2^-24 of sum p |v|, and 2^-140
where numbers end."""
import numpy as np
import pytest

import inputs
from test_gpu_attn_parts import run, setup

pytestmark = pytest.mark.gpu
LN2 = np.log(2.0)


def check(w, att, parent, n, p, with_ws=True):
    got = run(w, att, parent, n, p, with_ws)
    G, worst = w.Hq // w.Hkv, 0.0
    assert np.isfinite(got).all()
    for b in range(w.B):
        total = p[b] + n[b]
        sees = np.ones((n[b], total), bool)
        for i in range(n[b]):
            path, j = set(), i
            while j >= 0:
                path.add(j)
                j = int(parent[b, j])
            sees[i, p[b]:] = [j in path for j in range(n[b])]
        for h in range(w.Hkv):
            rows = lambda c: np.asarray(c)[att["block_table"][b], h].reshape(-1, w.D)[:total].astype(np.float64)
            k, v = rows(att["k_cache"][0]), rows(att["v_cache"][0])
            q = att["q"][0][b, :n[b], h * G:(h + 1) * G].astype(np.float64).reshape(-1, w.D)
            seen = np.repeat(sees, G, 0)
            s = np.where(seen, att["scale"] * (q @ k.T), -np.inf)
            m = s.max(-1, keepdims=True)
            e = np.exp(s - m)
            pr = e / e.sum(-1, keepdims=True)
            off = 29 * 2.0 ** -24 * att["scale"] * (np.abs(q) @ np.abs(k).T) + 4 * 2.0 ** -22 * np.maximum(LN2, np.abs(m))
            off = np.where(pr > 0, off, 0.0)
            a = (5 + 12 * (-(-total // 256) + 1) + 48) * 2.0 ** -24
            bound = (pr * (off + (pr * off).sum(-1, keepdims=True))) @ np.abs(v) + a * (pr @ np.abs(v)) + 2.0 ** -140
            err = np.abs(got[b, :n[b], h * G:(h + 1) * G].reshape(-1, w.D) - pr @ v)
            worst = max(worst, (err / bound).max())
    print("largest error / bound %.3f" % worst)
    assert worst <= 1.0


def arrays(D, P=2048, K=40):
    w, att, parent, rng = setup(1, K, 32, 8, D, P)
    return w, att, parent, rng, [np.array(att[x][0]) for x in ("q", "k_cache", "v_cache")], np.array([K], np.int32), np.array([P], np.int32)


def tokens(att, first, last):
    """Pages and slots of the tokens [first, last)."""
    t = np.arange(first, last)
    return att["block_table"][0, t // 16], t % 16


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("power", [16, 24, 40, 90])
@pytest.mark.parametrize("dims", ["all", "one"])
def test_values_of_a_node_that_few_rows_see(D, power, dims):
    """A node's values are far larger than all others'; its descendants see it, the rest of the tree does not."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    page, slot = (int(x[0]) for x in tokens(att, 2048 + 20, 2048 + 21))
    v[page, :, slot, slice(None) if dims == "all" else 5] *= np.float32(2.0 ** power)
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1e-5, 1e-8, 1e-30])
@pytest.mark.parametrize("dims", ["all", "one"])
def test_small_values_behind_zeros(D, size, dims):
    """The tokens that the wavefronts take first, the last 256, have values of zero in some dims, all others small ones there."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    d = slice(None) if dims == "all" else 7
    v[..., d] *= np.float32(size)
    for a, c in zip(*tokens(att, 2088 - 264, 2088)):
        v[a, :, c, d] = 0
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p, with_ws=False)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("power", [14, 20, 40])
def test_small_values_behind_large_ones_of_no_weight(D, power):
    """The tokens that the wavefronts take first have large values and scores so low that their weights vanish beside the others'."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    q[:] = q[0, 0, 0]
    low = q[0, 0, 0] * np.float32(-(60 + power) / (att["scale"] * (q[0, 0, 0].astype(np.float64) ** 2).sum()))
    for a, c in zip(*tokens(att, 2088 - 264, 2088)):
        k[a, :, c] = low
        v[a, :, c] *= np.float32(2.0 ** power)
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p, with_ws=False)


@pytest.mark.parametrize("D", [64, 128])
def test_values_near_the_smallest_numbers(D):
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v * np.float32(2.0 ** -118)]), parent, n, p)


@pytest.mark.parametrize("D", [64, 128])
def test_one_large_score_over_many_small_weights(D):
    """One key has nearly all of the weight; the others, 2^-26 of it each, keep theirs."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D, P=8500)
    q[:] = q[0, 0, 0]
    k[:] = 0
    a, c = (int(x[0]) for x in tokens(att, 300, 301))
    k[a, :, c] = q[0, 0, 0] * np.float32(26 * LN2 / (att["scale"] * (q[0, 0, 0].astype(np.float64) ** 2).sum()))
    v = np.abs(v)
    v[a, :, c] = 0
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p, with_ws=False)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-8])
@pytest.mark.parametrize("where", ["every_key", "one_key"])
def test_small_keys_beside_large_ones(D, size, where):
    """One dim of the keys, of every one or of one in a tile, is large where the queries are nearly zero; the others are small, and the
    queries so large that the scores have ordinary sizes."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    q, k = q / np.float32(size), k * np.float32(size)
    q[..., 3] = rng.standard_normal(q.shape[:-1]) * 1e-3
    if where == "every_key":
        k[..., 3] = 4 + rng.random(k.shape[:-1])
    else:
        for a, c in zip(*tokens(att, 0, 2088)):
            k[a, :, c, 3] = 4.5 if c == 9 else 0
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("power", [10, 16, 24, 40])
@pytest.mark.parametrize("only", [None, 0, 3, 30, 61])
def test_small_queries_beside_a_large_one(D, power, only):
    """A row's largest query by far meets keys of zero; keys that are zero but in one dim, too."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    if only is not None:
        k[..., [d for d in range(D) if d != only]] = 0
    q[..., 11] = np.float32(2.0 ** power)
    k[..., 11] = 0
    check(w, dict(att, q=[q], k_cache=[k], v_cache=[v]), parent, n, p)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("what", ["queries", "keys"])
def test_scores_of_the_smallest_and_largest_numbers(D, what):
    """Queries of 2^-110 with keys of 2^110, and the other way round: past what the factors reach."""
    w, att, parent, rng, (q, k, v), n, p = arrays(D)
    f = np.float32(2.0 ** (-110 if what == "queries" else 110))
    check(w, dict(att, q=[q * f], k_cache=[k / f], v_cache=[v]), parent, n, p)
