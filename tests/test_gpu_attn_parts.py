"""GPU parity of the fp32 attention kernel that multiplies on the 16-bit matrix cores, where its tiles, factors and second pass can go
wrong, against the CPU oracle (MI355X only).

Bound of a result in dim d, |error| <= (2 s + a) sum_t p_t |v_td|.  s, a score's error: its operands keep 23 bits (2^-23 each, one
partial product of 2^-24 left out), and its 24 partial sums are rounded to fp32 (2^-24 of at most sum |q k| <= |q| |k|), so s = (2.5 * 2^-23
+ 24 * 2^-24) scale max|q| max|k|, and a weight is off by a factor e^(2 s).  a: up to 2^-22 of a
product of probability and value is left out, and a sum is rounded twelve times a tile (six are allowed for: roundings are of either
sign) and once a wavefront, split and merge: (5 + 6 tiles + 48) 2^-24."""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2605_20104_amd as graft
from gpu_util import attn_plan, dev, host, widened
from test_gpu_attn import gpu_mask, shape_workload

pytestmark = pytest.mark.gpu


def run(w, att, parent, n, p, with_ws=True):
    assert attn_plan(w.B, w.K, w.Hq, w.Hkv, w.D, att["block_table"].shape[1], "f32").kernel == "tree_attn_parts_kernel"
    out = torch.full((w.B, w.K, w.Hq, w.D), 7.0, device="cuda")
    graft.graft_tree_attn(dev(att["q"][0], "f32"), dev(att["k_cache"][0], "f32"), dev(att["v_cache"][0], "f32"), att["strides"],
                          dev(att["block_table"]), dev(p), dev(n), gpu_mask(parent, n, p), w.Hkv, att["scale"], out=out,
                          workspace=None if with_ws else torch.empty(0, dtype=torch.uint8, device="cuda"))
    return host(out).astype(np.float64)


def reference(w, att, parent, n, p, rows=None):
    """The oracle's rows and their bounds."""
    f = lambda v: oracle.tree_attn(att["q"][0], att["k_cache"][0], v, "f32", att["strides"], att["block_table"], p, n, parent, w.Hq, w.Hkv,
                                   w.D, 16, att["scale"], rows=rows)
    norm = lambda x: np.sqrt((x.astype(np.float64) ** 2).sum(-1)).max()
    s = (2.5 * 2.0 ** -23 + 24 * 2.0 ** -24) * att["scale"] * norm(att["q"][0]) * norm(att["k_cache"][0])
    a = (5 + 6 * (-(-(w.P + w.K) // 256) + 1) + 48) * 2.0 ** -24
    return f(att["v_cache"][0]), (np.expm1(2 * s) + a) * f(np.abs(att["v_cache"][0]))


def setup(B, K, Hq, Hkv, D, P, layout="head_major", pages=0, seed=0):
    w = shape_workload(B, K, Hq, Hkv, D, P, dtype="f32")
    att = inputs.make_attention_inputs(w, seed=P + K + seed, layout=layout)
    rng = np.random.default_rng(P + K + seed)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    return w, (widened(att, pages) if pages else att), parent, rng


# lengths around tiles of 32 keys and around the eight wavefronts' first tiles (the table has room for more: wavefronts without a tile),
# rows off the tiles of 32, splits; without a workspace, which leaves the keys unsplit, more tiles a wavefront than the table register holds (32)
CASES = [
    (128, 4, 24, 32, 8, 0, "head_major", 320, True), (128, 4, 24, 32, 8, 7, "token_major", 320, True), (128, 4, 24, 32, 8, 8, "head_major", 320, True),
    (128, 4, 24, 32, 8, 9, "head_major", 320, True),
    (128, 1, 40, 32, 8, 215, "head_major", 130, True), (128, 1, 40, 32, 8, 216, "head_major", 130, True), (128, 1, 40, 32, 8, 217, "token_major", 130, True),
    (128, 1, 40, 32, 8, 2048, "head_major", 0, True), (128, 3, 57, 16, 2, 800, "token_major", 0, True), (128, 16, 24, 8, 8, 1000, "head_major", 0, True),
    (128, 1, 128, 32, 2, 900, "head_major", 0, True), (128, 1, 40, 32, 8, 8500, "head_major", 0, False), (128, 2, 33, 64, 4, 5000, "head_major", 0, True),
    (64, 1, 40, 32, 8, 2047, "head_major", 0, True), (64, 2, 61, 16, 4, 5000, "token_major", 0, True), (64, 4, 64, 32, 8, 33, "head_major", 96, True),
    (64, 1, 33, 16, 2, 9000, "head_major", 0, False),
    # a last tile of one token, which a wavefront takes first
    (128, 1, 40, 32, 8, 2009, "head_major", 0, False), (64, 2, 33, 16, 2, 4064, "token_major", 0, False), (128, 5, 126, 18, 2, 611, "head_major", 0, True),
    # tables of fewer than 48 pages with D = 128: 30 pages and one row group of the other kernel's, four steps a compute unit
    (128, 1, 121, 56, 4, 346, "head_major", 0, True), (128, 1, 70, 20, 2, 581, "token_major", 0, True), (128, 15, 52, 26, 2, 438, "head_major", 0, True),
    (128, 14, 43, 60, 4, 240, "token_major", 0, False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "D%d_B%d_K%d_Hq%d_Hkv%d_P%d_%s_%d_%s" % c)
def test_tiles_and_splits(case):
    D, B, K, Hq, Hkv, P, layout, pages, with_ws = case
    w, att, parent, rng = setup(B, K, Hq, Hkv, D, P, layout, pages)
    n, p = np.full(B, K, np.int32), np.full(B, P, np.int32)
    if B > 1:                                                  # ragged: fewer nodes, shorter prefixes, one absent tree
        n[1:], p[1:] = rng.integers(1, K + 1, B - 1), rng.integers(0, P + 1, B - 1)
        n[-1] = 0 if B > 2 else n[-1]
    got = run(w, att, parent, n, p, with_ws)
    assert np.isfinite(got).all()
    for b in range(B):
        assert (got[b, n[b]:] == 0).all()
    rows = None
    if B * K * Hq * (P + K) > 3_000_000:                       # a sample that has the first and the last row of every sequence
        rows = [(b, int(rng.integers(K)), int(rng.integers(Hq))) for b in range(B) for _ in range(24)]
        rows += [(b, i, h) for b in range(B) for i in (0, K - 1) for h in (0, Hq - 1)]
    ref, bound = reference(w, att, parent, n, p, rows)
    err = np.abs((got if rows is None else np.stack([got[r] for r in rows])) - ref)
    print("largest error / bound %.3f" % (err / np.maximum(bound, 1e-300)).max())
    assert (err <= bound).all()
    assert np.linalg.norm(err) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("what", ["small", "large", "dims", "keys_grow", "values_grow", "past_fp16"])
def test_magnitudes(D, what):
    """Sizes: all operands small or large (with the scores as they were), dims of values 2^-20 to 2^20 apart, keys and values that grow or
    shrink along the sequence, keys that no fp16 number holds."""
    w, att, parent, rng = setup(2, 40, 32, 8, D, 1500)
    n, p = np.array([40, 23], np.int32), np.array([1500, 1111], np.int32)
    q, k, v = (np.array(att[x][0]) for x in ("q", "k_cache", "v_cache"))
    f32 = np.float32
    if what == "small":
        q, k, v = q * f32(2.0 ** 12), k * f32(2.0 ** -12), v * f32(2.0 ** -60)
    elif what == "large":
        q, k, v = q * f32(2.0 ** -9), k * f32(2.0 ** 9), v * f32(2.0 ** 60)
    elif what == "dims":
        v = v * np.exp2(rng.integers(-20, 21, D)).astype(f32)
    elif what == "past_fp16":
        q, k = q * f32(2.0 ** -17), k * f32(2.0 ** 17)
    else:
        step = np.exp2(np.round(np.linspace(-13, 2 if what == "keys_grow" else 6, att["block_table"].shape[1]))).astype(f32)
        for b in range(2):
            x = k if what == "keys_grow" else v
            x[att["block_table"][b]] *= (step if b == 0 else step[::-1]).reshape((-1,) + (1,) * (x.ndim - 1))
    att = dict(att, q=[q], k_cache=[k], v_cache=[v])
    got = run(w, att, parent, n, p)
    ref, bound = reference(w, att, parent, n, p)
    err = np.abs(got - ref)
    print("largest error / bound %.3f" % (err / np.maximum(bound, 1e-300)).max())
    assert (err <= bound).all()


@pytest.mark.parametrize("D", [64, 128])
def test_keys_that_are_not_finite(D):
    """An infinite or NaN key counts only for the rows that see it: a score of -inf is a weight of zero, NaN makes a row's sum NaN, which
    the merge takes for a row without one (zeros, as from the fp32 MFMAs)."""
    B, K, Hq, Hkv, P = 1, 40, 32, 8, 1500
    w, att, parent, _ = setup(B, K, Hq, Hkv, D, P)
    parent = np.maximum(np.arange(K, dtype=np.int32)[None] - 1, -1)      # a chain: node i sees the slots up to i
    n, p = np.full(B, K, np.int32), np.full(B, P, np.int32)
    q, k = np.abs(att["q"][0]) + np.float32(0.5), np.array(att["k_cache"][0])
    att = dict(att, q=[q], k_cache=[k])
    clean = run(w, att, parent, n, p)
    at = lambda slot: (int(att["block_table"][0, (P + slot) // 16]), slice(None), (P + slot) % 16, 5)
    bad = k.copy()
    bad[at(30)] = np.nan
    got = run(w, dict(att, k_cache=[bad]), parent, n, p)
    assert (got[0, 30:] == 0).all()
    assert np.abs(got[0, :30] - clean[0, :30]).max() <= 2e-5           # (the second pass rounds elsewhere: as test_direct_path's fp32)
    bad = k.copy()
    bad[at(30)] = -np.inf                                              # the same as a key of which nothing is left
    none = k.copy()
    none[at(30)] = -1e30
    got, want = run(w, dict(att, k_cache=[bad]), parent, n, p), run(w, dict(att, k_cache=[none]), parent, n, p)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= 2e-5


@pytest.mark.parametrize("D", [64, 128])
def test_small_values_behind_large_ones(D):
    """Rows that see one token whose values are 2^-9 of all others': at most 2^-22 of their products is left out (2.4e-7), beside the
    sums' roundings."""
    w, att, parent, rng = setup(1, 40, 32, 8, D, 1500)
    n, p, t = np.array([40], np.int32), np.array([1500], np.int32), 300
    q, k, v = (np.array(att[x][0]) for x in ("q", "k_cache", "v_cache"))
    q[:] = q[0, 0, 0]
    page = att["block_table"][0, t // 16]
    k[page, :, t % 16] = q[0, 0, 0] * np.float32(60 / (att["scale"] * (q[0, 0, 0].astype(np.float64) ** 2).sum()))
    small = v[page, :, t % 16].copy()
    v *= np.float32(512)
    v[page, :, t % 16] = small
    att = dict(att, q=[q], k_cache=[k], v_cache=[v])
    got = run(w, att, parent, n, p)
    ref, _ = reference(w, att, parent, n, p)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("relative error %.2e" % rel)
    assert rel <= 5e-7
