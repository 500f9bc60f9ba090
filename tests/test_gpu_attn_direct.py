"""GPU parity of the attention path for fp32 storage and for bf16 with head size 64, at the sizes
where its tiling can go wrong, against the CPU oracle (MI355X only).

Bounds.  fp32: 1e-4, as for every fp32 case.  bf16: scores, softmax, probabilities and sums are
fp32, so what is left is the rounding of the result to bf16: 8 significant
bits, so at most 2^-8 of the value (half of the spacing 2^-7 right above a power of two), plus 1e-4
for everything before it."""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2605_20104_amd as graft
from gpu_util import attn_plan, dev, host, widened
from test_gpu_attn import check_case, gpu_mask, shape_workload

pytestmark = pytest.mark.gpu

# (dtype, D, B, K, Hq, Hkv, P, layout, workspace): tiles are 32 keys (bf16) or 16 (fp32)
CASES = [
    ("f32", 64, 1, 1, 1, 1, 0, "head_major", True),            # a lone root, empty prefix
    ("f32", 128, 1, 1, 2, 1, 15, "head_major", True),          # exactly one tile
    ("f32", 128, 1, 2, 2, 1, 15, "token_major", True),         # one key more
    ("f32", 64, 2, 17, 6, 2, 300, "head_major", True),         # rows and keys off every boundary
    ("f32", 128, 1, 40, 32, 8, 1000, "head_major", True),
    ("f32", 128, 2, 128, 32, 2, 90, "head_major", True),       # 2048 rows: the most row tiles, both mask words
    ("f32", 64, 1, 4, 1, 1, 9000, "head_major", False),        # one workgroup for all keys: a wavefront walks many tiles
    ("f32", 128, 3, 9, 4, 4, 2500, "token_major", False),
    ("bf16", 64, 1, 1, 1, 1, 0, "head_major", True),
    ("bf16", 64, 1, 1, 4, 4, 31, "head_major", True),
    ("bf16", 64, 1, 2, 4, 4, 31, "token_major", True),
    ("bf16", 64, 2, 33, 8, 2, 700, "head_major", True),
    ("bf16", 64, 1, 60, 32, 8, 2048, "token_major", True),
    ("bf16", 64, 4, 128, 16, 1, 500, "head_major", True),      # 2048 rows
    ("bf16", 64, 1, 3, 2, 1, 9001, "head_major", False),
    ("bf16", 64, 16, 24, 16, 8, 333, "head_major", True),      # enough units for one split
    ("bf16", 64, 1, 64, 16, 2, 12000, "head_major", True),     # many splits, wide row tiles
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_D%d_B%d_K%d_Hq%d_Hkv%d_P%d_%s_%s" % c)
def test_direct_path(case):
    dtype, D, B, K, Hq, Hkv, P, layout, with_ws = case
    w = shape_workload(B, K, Hq, Hkv, D, P, dtype=dtype)
    rng = np.random.default_rng(P + K)
    att = inputs.make_attention_inputs(w, seed=P + K, layout=layout)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    n_nodes, prefix = np.full(B, K, np.int32), np.full(B, P, np.int32)
    if B > 1:                                                  # ragged: fewer nodes, shorter prefixes, one absent tree
        n_nodes[1:] = rng.integers(1, K + 1, B - 1)
        prefix[1:] = rng.integers(0, P + 1, B - 1)
        n_nodes[-1] = 0 if B > 2 else n_nodes[-1]
    mask = gpu_mask(parent, n_nodes, prefix)
    ws = None if with_ws else torch.empty(0, dtype=torch.uint8, device="cuda")
    out = torch.full((B, K, Hq, D), 7.0, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    graft.graft_tree_attn(dev(att["q"][0], dtype), dev(att["k_cache"][0], dtype), dev(att["v_cache"][0], dtype), att["strides"],
                          dev(att["block_table"]), dev(prefix), dev(n_nodes), mask, Hkv, att["scale"], out=out, workspace=ws)
    got = host(out).astype(np.float64)
    rows = None
    if B * K * Hq * (P + K) > 3_000_000:                       # a sample that has the first and the last row of every sequence
        rows = [(b, int(rng.integers(K)), int(rng.integers(Hq))) for b in range(B) for _ in range(24)]
        rows += [(b, i, h) for b in range(B) for i in (0, K - 1) for h in (0, Hq - 1)]
    ref = oracle.tree_attn(att["q"][0], att["k_cache"][0], att["v_cache"][0], dtype, att["strides"], att["block_table"], prefix,
                           n_nodes, parent, Hq, Hkv, D, 16, att["scale"], rows=rows)
    sel = got if rows is None else np.stack([got[r] for r in rows])
    bound = 1e-4 + (0.0 if dtype == "f32" else 2.0 ** -8) * np.abs(ref)
    err = np.abs(sel - ref)
    assert np.isfinite(got).all()
    assert (err <= bound).all(), "error %.3e, bound there %.3e" % (err.max(), bound.flat[(err - bound).argmax()])
    for b in range(B):
        assert (got[b, n_nodes[b]:] == 0).all()                # rows of absent nodes


# Wavefronts with several 16-row blocks: bf16 in blocks of 32 rows through the 32x32 products, fp32 with D = 128 with queries
# shared through LDS where a row group has several wavefronts.  (case, row blocks, row groups, whether the keys are split
# over workgroups); 33 x 16, 50, 24 and 60 x 4 rows are no multiples of 32.
ROW_BLOCKS = [
    (("bf16", 64, 4, 60, 32, 8, 2048, "token_major", True), 2, 1, False),
    (("bf16", 64, 4, 33, 64, 4, 700, "head_major", True), 2, 2, False),
    (("bf16", 64, 3, 128, 64, 4, 100, "head_major", True), 2, 4, False),
    (("bf16", 64, 6, 97, 64, 4, 100, "token_major", True), 2, 8, False),
    (("bf16", 64, 3, 50, 8, 8, 5000, "head_major", True), 2, 1, True),
    (("bf16", 64, 6, 24, 8, 8, 5000, "head_major", True), 2, 1, True),
    (("bf16", 64, 4, 33, 64, 4, 2048, "head_major", True), 2, 4, True),
    (("bf16", 64, 2, 128, 64, 4, 3000, "head_major", True), 4, 1, False),
    (("bf16", 64, 4, 33, 64, 4, 1500, "token_major", True), 4, 1, False),
    (("bf16", 64, 8, 33, 64, 4, 700, "head_major", True), 4, 2, False),
    (("bf16", 64, 8, 79, 64, 4, 300, "head_major", True), 4, 4, False),
    (("bf16", 64, 2, 33, 64, 4, 5000, "head_major", True), 4, 1, True),
    (("bf16", 64, 6, 97, 32, 8, 5000, "head_major", True), 4, 8, True),
    (("f32", 128, 4, 33, 32, 8, 700, "head_major", True), 2, 1, False),
    (("f32", 128, 6, 128, 12, 4, 100, "token_major", True), 2, 2, False),
    (("f32", 128, 2, 33, 64, 4, 700, "head_major", True), 2, 2, True),
    (("f32", 128, 4, 33, 64, 4, 700, "head_major", True), 2, 4, True),
    (("f32", 128, 3, 97, 64, 4, 300, "head_major", True), 2, 8, True),
]


@pytest.mark.parametrize("case,row_blocks,row_groups,split", ROW_BLOCKS, ids=lambda x: "%s_D%d_B%d_K%d_Hq%d_Hkv%d_P%d_%s_%s" % x if isinstance(x, tuple) else str(x))
def test_several_row_blocks(case, row_blocks, row_groups, split):
    dtype, D, B, K, Hq, Hkv, P, _, _ = case
    plan = attn_plan(B, K, Hq, Hkv, D, (P + K + 15) // 16, dtype)
    blocks = (K * (Hq // Hkv) + 15) // 16
    assert (plan.path, plan.row_blocks, plan.splits > 1) == ("direct", row_blocks, split)
    assert plan.row_tiles == -(-blocks // (row_groups * row_blocks))       # as many as that many row groups leave
    test_direct_path(case)


@pytest.mark.parametrize("dtype,D,B,K,Hq,Hkv,row_blocks", [("f32", 64, 1, 24, 4, 2, 1), ("f32", 128, 1, 24, 4, 2, 1), ("bf16", 64, 1, 24, 4, 2, 1),
                                                           ("bf16", 64, 2, 33, 64, 4, 2), ("f32", 128, 2, 33, 64, 4, 2)])
def test_scores_that_keep_rising(dtype, D, B, K, Hq, Hkv, row_blocks):
    """Scores rising by far more than the lazy bound along the sequence: the reference is raised again and
    again; falling scores keep the first one.  Bound: a dot product of D equal terms summed in fp32 is off by
    at most D/2 * 2^-24 of itself (D partial sums, half of the full one on average), which moves a weight by
    that fraction of the largest score and the result by as much times the largest |v|; plus, for bf16, the
    rounding of the result."""
    assert attn_plan(B, K, Hq, Hkv, D, (1500 + K + 15) // 16, dtype).row_blocks == row_blocks
    w = shape_workload(B, K, Hq, Hkv, D, 1500, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=3)
    conv = (lambda a: a) if dtype == "f32" else inputs.bf16_bits_to_f32
    back = (lambda a: a.astype(np.float32)) if dtype == "f32" else inputs.f32_to_bf16_bits
    k, q = conv(att["k_cache"][0]).copy(), conv(att["q"][0]).copy()
    for lp in range(att["pages_per_seq"]):
        t = lp * 16 + np.arange(16)
        k[att["block_table"][:, lp]] = (t * 0.05)[None, :, None]
    q[:] = 1.0
    q[:, :, 1::2, :] = -1.0
    att["k_cache"], att["q"] = [back(k)], [back(q)]
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(3), w.K, 8)] * B)
    n, p = np.full(B, w.K, np.int32), np.full(B, w.P, np.int32)
    for ws in (None, torch.empty(0, dtype=torch.uint8, device="cuda")):
        out = graft.graft_tree_attn(dev(att["q"][0], dtype), dev(att["k_cache"][0], dtype), dev(att["v_cache"][0], dtype),
                                    att["strides"], dev(att["block_table"]), dev(p), dev(n), gpu_mask(parent, n, p), w.Hkv,
                                    att["scale"], workspace=ws)
        ref = oracle.tree_attn(att["q"][0], att["k_cache"][0], att["v_cache"][0], dtype, att["strides"], att["block_table"], p, n,
                               parent, w.Hq, w.Hkv, w.D, 16, att["scale"])
        err = np.abs(host(out).astype(np.float64) - ref)
        s_max = w.P * 0.05 * D * att["scale"]
        bound = D / 2 * 2.0 ** -24 * s_max * np.abs(conv(att["v_cache"][0])).max()
        print("largest score %.0f, bound %.1e, max error %.1e" % (s_max, bound, err.max()))
        assert (err <= bound + (0.0 if dtype == "f32" else 2.0 ** -8) * np.abs(ref)).all(), err.max()


# bf16 with D = 128 takes the direct path where the keys are few (the probabilities are rounded to bf16
# there, relative 2^-8 each with random sign, and so is the result: the 2e-2 of every D = 128 test)
@pytest.mark.parametrize("case", [(1, 1, 1, 1, 100), (1, 20, 8, 8, 300), (2, 33, 6, 2, 63), (1, 78, 8, 1, 37), (3, 128, 32, 2, 20),
                                  (8, 24, 32, 8, 500), (1, 40, 32, 8, 700)], ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d" % c)
@pytest.mark.parametrize("layout", ["head_major", "token_major"])
def test_head_128_with_few_keys(case, layout):
    B, K, Hq, Hkv, P = case
    assert attn_plan(B, K, Hq, Hkv, 128, (P + K + 15) // 16, "bf16").path == "direct"
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(K)
    n_nodes = None if B == 1 else np.concatenate([[K], rng.integers(1, K + 1, B - 1)]).astype(np.int32)
    prefix = None if B == 1 else np.concatenate([[P], rng.integers(0, P + 1, B - 1)]).astype(np.int32)
    check_case(w, seed=K + P, layout=layout, n_nodes=n_nodes, prefix=prefix)


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_tensors_that_start_at_any_element(dtype, D):
    """Rows are 16 bytes apart or a multiple of it, but a tensor may start at any element: the bits are those of the
    same data at the start of an allocation (the same path, hence the same order of every sum)."""
    w = shape_workload(1, 20, 8, 8, D, 100, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=9)
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(9), w.K, 8)])
    n, p = np.array([w.K], np.int32), np.array([w.P], np.int32)
    mask = gpu_mask(parent, n, p)
    tensors = [dev(att[k][0], dtype) for k in ("q", "k_cache", "v_cache")] + [torch.zeros_like(dev(att["q"][0], dtype))]

    def moved(t):
        u = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape)
        return u.copy_(t)

    def run(q, k, v, out):
        return graft.graft_tree_attn(q, k, v, att["strides"], dev(att["block_table"]), dev(p), dev(n), mask, w.Hkv, att["scale"], out=out)

    a, b = run(*tensors), run(*[moved(t) for t in tensors])
    assert torch.equal(a, b)


@pytest.mark.parametrize("K,G,H,pages,row_blocks", [(1, 1, 32, 1, 1), (3, 16, 32, 100, 2), (9, 16, 16, 200, 4)])
def test_probabilities_keep_their_32_bits_with_head_64(K, G, H, pages, row_blocks):
    """Values chosen so that the weighted sum all but cancels: what is left of it shows every bit a probability
    loses on its way into the product with the values.  Four keys, scores that fp32 holds exactly (queries and
    keys have one nonzero element), results far smaller than their terms.  Bound: the exponent x = (s - max) log2 e
    is below 16 with one rounding (16 * 2^-24 ln 2 of p) and exp2 is good to 2^-23, so a probability is off by at
    most 2^-20 of itself, four sums add 2^-22 of the terms; plus the rounding of the result.  Probabilities of
    17 bits are off by up to 2^-17."""
    B, D, P = 4, 64, 3
    assert attn_plan(B, K, G * H, H, D, pages, "bf16").row_blocks == row_blocks
    rng = np.random.default_rng(17)
    w = shape_workload(B, K, G * H, H, D, P)
    att = inputs.make_attention_inputs(w, seed=17)
    k, v = np.zeros_like(inputs.bf16_bits_to_f32(att["k_cache"][0])), np.zeros_like(inputs.bf16_bits_to_f32(att["v_cache"][0]))
    q = np.zeros((B, K, G * H, D), np.float32)
    q[..., 0] = 1.0
    bits = inputs.f32_to_bf16_bits
    round_bf16 = lambda a: inputs.bf16_bits_to_f32(bits(np.asarray(a, np.float32))).astype(np.float64)
    for b in range(B):
        page = att["block_table"][b, 0]
        s = round_bf16(rng.uniform(-6, 0, (H, 4)))
        p = np.exp(s - s.max(axis=1, keepdims=True))
        vals = np.zeros((H, 4, D))
        order = np.argsort(-p, axis=1)                         # each value cancels what the heavier keys leave, to 8 bits
        vals[np.arange(H), order[:, 0]] = round_bf16(rng.uniform(1, 2, (H, D)))
        for j in range(1, 4):
            at = order[:, j]
            left = np.einsum("ht,htd->hd", p, vals)
            vals[np.arange(H), at] = round_bf16(-left / p[np.arange(H), at][:, None])
        k[page, :, :4, 0] = s                                  # [page][head][token][dim]
        v[page, :, :4] = vals
    att["k_cache"], att["v_cache"], att["q"] = [bits(k)], [bits(v)], [bits(q)]
    # nodes below the root see a fifth key, their own, of score and value zero: it takes from all weights alike (and is a fifth
    # term of the sums, 2^-21 of the terms together)
    parent, n, prefix = np.zeros((B, K), np.int32), np.full(B, K, np.int32), np.full(B, P, np.int32)
    parent[:, 0] = -1
    att = widened(att, pages)
    out = graft.graft_tree_attn(dev(att["q"][0], "bf16"), dev(att["k_cache"][0], "bf16"), dev(att["v_cache"][0], "bf16"),
                                att["strides"], dev(att["block_table"]), dev(prefix), dev(n), gpu_mask(parent, n, prefix), H, 1.0)
    got = host(out).astype(np.float64)
    for b, i, member in [(b, i, j) for b in range(B) for i in range(K) for j in range(G)]:
        page = att["block_table"][b, 0]
        s, vals = k[page, :, :4, 0].astype(np.float64), v[page, :, :4].astype(np.float64)
        own = np.zeros(H) if i == 0 else np.exp(-s.max(axis=1))
        p = np.exp(s - s.max(axis=1, keepdims=True))
        p /= (p.sum(axis=1) + own)[:, None]
        ref, size = np.einsum("ht,htd->hd", p, vals), np.einsum("ht,htd->hd", p, np.abs(vals))
        err = np.abs(got[b, i, member::G] - ref)
        bound = (2.0 ** -20 + (2.0 ** -22 if i == 0 else 2.0 ** -21)) * size + 2.0 ** -8 * np.abs(ref)
        if member == 0:
            print("largest error / bound %.2f, median of result / terms %.1e" % ((err / bound).max(), np.median(np.abs(ref) / size)))
        assert (err <= bound).all(), (err / bound).max()


@pytest.mark.parametrize("dtype,D,K,Hq,P", [("f32", 64, 40, 8, 300), ("f32", 128, 23, 4, 77), ("f32", 128, 128, 64, 1500), ("bf16", 64, 40, 8, 300),
                                            ("bf16", 64, 128, 64, 3000), ("bf16", 64, 33, 64, 1500)])
def test_values_that_are_not_finite_stay_with_the_nodes_that_see_them(dtype, D, K, Hq, P):
    """Infinite and NaN values in tree slots, the last one among them: rows that do not see the slot are those of a run
    without them, rows that do get inf or NaN in that dim alone.  Bound: the walk that keeps such values out takes the exact
    running maximum as a row's reference, the other one may lag behind it, so the sums are rounded elsewhere: fp32 within
    1e-5, bf16 results within one unit in the last place, 2^-7."""
    B, Hkv = 2, 4
    w = shape_workload(B, K, Hq, Hkv, D, P, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=D + K)
    rng = np.random.default_rng(D + K)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    n, p = np.full(B, K, np.int32), np.full(B, P, np.int32)
    mask = gpu_mask(parent, n, p)
    words = host(mask)
    sees = np.array([[[int(words[b, i, j // 64]) >> (j % 64) & 1 for j in range(K)] for i in range(K)] for b in range(B)], bool)
    v = dev(att["v_cache"][0], dtype)                                      # [page][head][token][dim]
    planted = [(K - 1, 3, np.inf), (K // 2, 0, -np.inf), (K // 2, 5, np.nan), (1, D - 1, np.nan), (K // 3, 3, np.inf), (2, 5, -np.inf)]

    def run(values):
        return graft.graft_tree_attn(dev(att["q"][0], dtype), dev(att["k_cache"][0], dtype), values, att["strides"], dev(att["block_table"]),
                                     dev(p), dev(n), mask, Hkv, att["scale"])

    clean, bad = run(v), v.clone()
    touched = np.zeros((B, K), bool)
    want = np.zeros((B, K, D))                                             # inf, -inf or NaN where a seen value is
    for b in range(B):
        for slot, dim, x in planted:
            bad[int(att["block_table"][b, (P + slot) // 16]), :, (P + slot) % 16, dim] = float(x)
            touched[b] |= sees[b, :, slot]
            want[b, sees[b, :, slot], dim] += x
    got = run(bad)
    assert not touched.all()
    g, c = host(got).astype(np.float64), host(clean).astype(np.float64)
    want = np.broadcast_to(want[:, :, None], g.shape)
    odd = ~np.isfinite(want) | np.isnan(want)
    assert ((g == want) | (np.isnan(g) & np.isnan(want)))[odd].all()
    assert np.isfinite(g[~odd]).all()
    assert (np.abs(g - c)[~odd] <= (1e-5 if dtype == "f32" else 2.0 ** -7) * (1 + np.abs(c[~odd]))).all()


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("P,pages,with_ws", [(0, 3, True), (9, 40, True), (300, 22, True), (600, 200, True), (1500, 98, False), (17000, 1100, False)])
def test_entries_past_a_sequences_last_page_are_not_followed(dtype, D, P, pages, with_ws):
    check_unused_entries(dtype, D, 20, 2, 2, P, pages, with_ws)


@pytest.mark.parametrize("dtype,D,K,Hq,Hkv,P,pages,row_blocks", [
    ("bf16", 64, 33, 64, 4, 600, 200, 2), ("bf16", 64, 33, 64, 4, 1500, 98, 2), ("bf16", 64, 60, 32, 8, 2000, 130, 2),
    ("bf16", 64, 33, 64, 4, 17000, 1100, 4), ("f32", 128, 33, 64, 4, 9, 40, 2), ("f32", 128, 60, 32, 8, 2000, 130, 2)])
def test_entries_past_the_last_page_with_several_row_blocks(dtype, D, K, Hq, Hkv, P, pages, row_blocks):
    assert attn_plan(3, K, Hq, Hkv, D, pages, dtype).row_blocks == row_blocks
    check_unused_entries(dtype, D, K, Hq, Hkv, P, pages, True)


def check_unused_entries(dtype, D, K, Hq, Hkv, P, pages, with_ws):
    """Table entries are requested before the lengths are known.  Those behind a sequence's last page name a page of NaN
    here: the rows are those of a table that repeats the last page, bit for bit.  Splits that begin elsewhere than in a
    full table, wavefronts with more tiles than the request covers, an odd last page."""
    B = 3
    w = shape_workload(B, K, Hq, Hkv, D, P, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=P + 1)
    n, p = np.array([K, 0, 7], np.int32), np.array([P, P, P // 2], np.int32)
    used = att["block_table"].shape[1]
    assert pages >= used
    spare = np.setdiff1d(np.arange(len(att["k_cache"][0])), att["block_table"].ravel())
    assert len(spare) > 0
    caches = [dev(att[x][0], dtype).clone() for x in ("k_cache", "v_cache")]
    for c in caches:
        c[int(spare[0])] = float("nan")
    mask = gpu_mask(np.arange(-1, K - 1, dtype=np.int32)[None].repeat(B, 0), n, p)
    out = []
    for poison in (False, True):
        table = np.zeros((B, pages), np.int32)
        table[:, :used] = att["block_table"]
        for b in range(B):
            last = (p[b] + n[b] - 1) // 16 if n[b] else -1
            table[b, last + 1:] = spare[0] if poison else table[b, max(last, 0)]
        out.append(graft.graft_tree_attn(dev(att["q"][0], dtype), *caches, att["strides"], dev(table), dev(p), dev(n), mask, Hkv, att["scale"],
                                         workspace=None if with_ws else torch.empty(0, dtype=torch.uint8, device="cuda")
                                         if (dtype, D) != ("bf16", 128) else None))
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dtype,D,P,pages", [("bf16", 64, 170, 11), ("bf16", 64, 176, 11), ("bf16", 64, 200, 11), ("bf16", 128, 170, 11),
                                             ("bf16", 128, 8330, 521), ("f32", 64, 170, 11)])
def test_tree_slots_past_the_block_table_do_not_count(dtype, D, P, pages):
    """A tree that does not fit its table (an odd number of pages, so that the last tile of 32 or 64 keys reaches past it)
    is cut at the capacity: no token counts twice."""
    K, H = 24, 2
    w = shape_workload(1, K, H, H, D, pages * 16 - K, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=P)
    assert att["block_table"].shape[1] == pages
    assert attn_plan(1, K, H, H, D, pages, dtype).path == ("mfma" if pages > 500 else "direct")
    parent = np.arange(-1, K - 1, dtype=np.int32)[None]                    # a chain: every node sees all slots before it
    n, p = np.array([K], np.int32), np.array([P], np.int32)
    out = graft.graft_tree_attn(*(dev(att[x][0], dtype) for x in ("q", "k_cache", "v_cache")), att["strides"], dev(att["block_table"]), dev(p),
                                dev(n), gpu_mask(parent, n, p), H, att["scale"])
    f = (lambda a: a.astype(np.float64)) if dtype == "f32" else (lambda a: inputs.bf16_bits_to_f32(a).astype(np.float64))
    q, k, v = (f(att[x][0]) for x in ("q", "k_cache", "v_cache"))
    k, v = (x[att["block_table"][0]].transpose(1, 0, 2, 3).reshape(H, pages * 16, D) for x in (k, v))
    got = host(out).astype(np.float64)
    for i in range(K):
        seen = min(P + i + 1, pages * 16)
        for h in range(H):
            s = k[h, :seen] @ q[0, i, h] * att["scale"]
            e = np.exp(s - s.max())
            ref = e @ v[h, :seen] / e.sum()
            bound = 1e-4 if dtype == "f32" else (2e-2 if D == 128 else 1e-4 + 2.0 ** -8 * np.abs(ref))
            assert (np.abs(got[0, i, h] - ref) <= bound).all(), (i, h, np.abs(got[0, i, h] - ref).max())


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_queries_of_absent_nodes_may_be_anything(dtype, D):
    """NaN and infinities in the query rows behind n_nodes: the other rows keep their bits, these are zeros."""
    w = shape_workload(2, 33, 8, 2, D, 300, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=5)
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(b), w.K, 8) for b in range(w.B)])
    n, p = np.array([20, 33], np.int32), np.array([300, 117], np.int32)
    mask = gpu_mask(parent, n, p)
    q = dev(att["q"][0], dtype)
    wild = q.clone()
    wild[0, 20::2], wild[0, 21::2] = float("nan"), float("inf")
    clean, got = (graft.graft_tree_attn(x, dev(att["k_cache"][0], dtype), dev(att["v_cache"][0], dtype), att["strides"],
                                        dev(att["block_table"]), dev(p), dev(n), mask, w.Hkv, att["scale"]) for x in (q, wild))
    assert torch.equal(clean, got) and bool((got[0, 20:] == 0).all())


def test_first_call_inside_a_capture_with_more_than_64_kb_of_lds():
    """The opt-in for more LDS than the default limit comes with a host thread's first such launch: here that is inside a
    capture.  Every replay gives the bits of an eager call, with eager work in between."""
    import threading
    w = shape_workload(2, 40, 16, 4, 128, 600, dtype="f32")
    plan = attn_plan(w.B, w.K, w.Hq, w.Hkv, w.D, (w.P + w.K + 15) // 16, "f32")
    assert plan.path == "direct" and 8 * 16 * w.D * 4 >= 65536          # the staged keys alone; with the merge more
    att = inputs.make_attention_inputs(w, seed=2)
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(2), w.K, 8) for _ in range(w.B)])
    n, p = np.full(w.B, w.K, np.int32), np.full(w.B, w.P, np.int32)
    args = [dev(att[x][0], "f32") for x in ("q", "k_cache", "v_cache")] + [att["strides"], dev(att["block_table"]), dev(p), dev(n),
                                                                           gpu_mask(parent, n, p), w.Hkv, att["scale"]]
    eager = graft.graft_tree_attn(*args)
    out = torch.zeros_like(eager)
    need = graft.graft_tree_attn_workspace_bytes(w.B, w.K, w.Hq, w.Hkv, w.D, args[4].shape[1], graft.GRAFT_F32)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    g, failed = torch.cuda.CUDAGraph(), []

    def capture():
        try:
            with torch.cuda.graph(g):
                graft.graft_tree_attn(*args, out=out, workspace=ws)
        except Exception as e:                                            # shown below, in the test's thread
            failed.append(e)

    torch.cuda.synchronize()
    t = threading.Thread(target=capture)
    t.start()
    t.join()
    assert not failed, failed
    for _ in range(4):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        assert torch.equal(graft.graft_tree_attn(*args), eager)


def test_shapes_that_take_turns_on_one_thread():
    """Calls of ten shapes in turn, more than a thread keeps plans of, with and without a workspace: the bits of the first
    time, every time."""
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    calls = []
    for i, (dtype, D) in enumerate([("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128), ("bf16", 64)] * 2):
        w = shape_workload(1 + i % 3, 12 + 5 * i, 8, 2, D, 300 + 170 * i, dtype=dtype)
        att = inputs.make_attention_inputs(w, seed=i)
        parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(i), w.K, 8) for _ in range(w.B)])
        n, p = np.full(w.B, w.K, np.int32), np.full(w.B, w.P, np.int32)
        args = [dev(att[x][0], dtype) for x in ("q", "k_cache", "v_cache")] + [att["strides"], dev(att["block_table"]), dev(p), dev(n),
                                                                               gpu_mask(parent, n, p), w.Hkv, att["scale"]]
        calls += [(args, None)] + ([(args, none)] if (dtype, D) != ("bf16", 128) else [])
    first = [graft.graft_tree_attn(*a, workspace=ws) for a, ws in calls]
    for _ in range(3):
        for (a, ws), want in zip(calls, first):
            assert torch.equal(graft.graft_tree_attn(*a, workspace=ws), want)


def test_more_workgroups_than_one_launch_holds():
    """65535 sequences of 130 heads, one node each: 8.5 million workgroups of 512 threads, and a launch holds fewer than 2^32
    work-items.  All sequences share one page; every row is checked."""
    B, H, D, P = 65535, 130, 64, 3
    gen = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn((B, 1, H, D), generator=gen, device="cuda", dtype=torch.bfloat16)
    k, v = (torch.randn((1, H, 16, D), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    ints = lambda x: torch.full((B,), x, dtype=torch.int32, device="cuda")
    mask = torch.tensor([1, 0], dtype=torch.int64, device="cuda").expand(B, 1, 2).contiguous()
    out = graft.graft_tree_attn(q, k, v, {"page": H * 16 * D, "token": D, "head": 16 * D}, torch.zeros((B, 1), dtype=torch.int32, device="cuda"),
                                ints(P), ints(1), mask, H, 0.125)
    for h in range(H):
        kk, vv = k[0, h, :P + 1].float(), v[0, h, :P + 1].float()
        ref = torch.softmax(q[:, 0, h].float() @ kk.T * 0.125, -1) @ vv
        err = (out[:, 0, h].float() - ref).abs()
        assert bool((err <= 1e-4 + 2.0 ** -8 * ref.abs()).all()), (h, float(err.max()))


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_values_near_the_top_of_the_range(dtype, D):
    """Values of 2^118 under scores that lie 15 (in log2 units) above those of the keys taken first, too little for a row to
    raise its reference: a weight of 2^15 relative to that reference must not overflow.  All values are equal, so
    every row is that value."""
    K, H, P = 12, 2, 500
    w = shape_workload(1, K, H, H, D, P, dtype=dtype)
    att = inputs.make_attention_inputs(w, seed=4)
    back = (lambda a: a.astype(np.float32)) if dtype == "f32" else inputs.f32_to_bf16_bits
    q, k, v = (np.zeros(att[x][0].shape, np.float32) for x in ("q", "k_cache", "v_cache"))
    q[..., 0] = 1.0
    for lp in range(att["pages_per_seq"]):
        k[att["block_table"][0, lp], :, :, 0] = np.where(lp * 16 + np.arange(16) < 300, 15 * 0.6931, 0.0)
    v[:] = 2.0 ** 118
    parent, n, p = np.arange(-1, K - 1, dtype=np.int32)[None], np.array([K], np.int32), np.array([P], np.int32)
    for ws in (None, torch.empty(0, dtype=torch.uint8, device="cuda")):
        out = graft.graft_tree_attn(*(dev(back(x), dtype) for x in (q, k, v)), att["strides"], dev(att["block_table"]), dev(p), dev(n),
                                    gpu_mask(parent, n, p), H, 1.0, workspace=ws)
        got = host(out).astype(np.float64) / 2.0 ** 118
        assert (np.abs(got - 1) <= (1e-5 if dtype == "f32" else 2.0 ** -8)).all(), got.ravel()[:8]
