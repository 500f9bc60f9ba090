"""GPU parity of the MFMA attention kernel with 32-row blocks (tiles of 192, 256 and 384 rows, reported as 3, 4 and 6 times 64)
against the CPU oracle, at the edges of its tiles, of its score range and of its page table (MI355X only).  Every test asserts
that the shape takes this kernel.

Tolerance as for every bf16 test with D = 128: 2e-2 (test_gpu_attn.py says where it comes from)."""
import numpy as np
import pytest

import inputs
from gpu_util import attn_plan
from test_gpu_attn import TOL_BF16, score_scale_tolerance, shape_workload
from test_gpu_attn_mfma import compare, reference, run, sample

pytestmark = pytest.mark.gpu


def trees(rng, B, K):
    return np.stack([inputs.random_recursive_tree(rng, K, 8 if b % 2 else K - 1) for b in range(B)])


def assert_wide(plan, tile, split):
    assert (plan.kernel, plan.row_blocks, plan.splits > 1) == ("tree_attn_wide_kernel", tile, split), plan


# (B, K, Hq, Hkv, P, tile rows / 64, keys split over workgroups): with and without a last tile that is full
SHAPES = [(8, 60, 64, 4, 650, 3, False), (8, 80, 64, 4, 653, 3, False), (2, 72, 24, 2, 8000, 3, True), (2, 96, 64, 8, 3000, 3, True),
          (16, 100, 32, 2, 650, 4, False), (1, 100, 16, 1, 5000, 4, True), (8, 65, 32, 2, 503, 4, True), (1, 127, 16, 1, 5003, 4, True),
          (16, 96, 64, 4, 650, 6, False), (3, 96, 48, 4, 5000, 6, True), (6, 95, 24, 2, 5003, 6, True)]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_tile%d_split%d" % c)
@pytest.mark.parametrize("layout", ["head_major", "token_major"])
def test_tiles(case, layout):
    """Ragged prefixes and trees: rows of absent nodes in and behind a tile, lengths off every boundary of a page, a sub-tile
    and a stage, splits with one stage less than others or none, one sequence that is absent."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(P + K)
    att = inputs.make_attention_inputs(w, seed=P + K, layout=layout)
    parent = trees(rng, B, K)
    n_nodes, prefix = np.full(B, K, np.int32), np.full(B, P, np.int32)
    n_nodes[1:], prefix[1:] = rng.integers(1, K + 1, B - 1), rng.integers(0, P + 1, B - 1)
    if B > 4:
        n_nodes[2], prefix[3] = 0, 0
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1))


@pytest.mark.parametrize("case", [SHAPES[2], SHAPES[3], SHAPES[6], SHAPES[9], (8, 48, 64, 4, 4096, 3, True)],
                         ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_tile%d_split%d" % c)
@pytest.mark.parametrize("long_one", [False, True], ids=["all_short", "one_long"])
def test_splits_without_a_stage(case, long_one):
    """Sequences far shorter than their block table: workgroups whose split has no keys hand on empty rows, whatever the
    queries that they have requested hold."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(P + K + 1)
    att = inputs.make_attention_inputs(w, seed=P + K + 1)
    parent = trees(rng, B, K)
    n_nodes, prefix = rng.integers(1, K + 1, B).astype(np.int32), rng.integers(0, 64, B).astype(np.int32)
    if long_one:
        n_nodes[0], prefix[0] = K, P
    q = att["q"][0].copy()
    for b in range(B):
        q[b, n_nodes[b]:] = 0x7f80
    att["q"] = [q]
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    assert min(-(-(prefix + n_nodes) // 64)) < plan.splits
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 120 // B + 1))


def scored(w, att, level):
    """Queries of ones and keys that give every row the score level(sequence, token), in natural units; odd heads get it negated."""
    k = inputs.bf16_bits_to_f32(att["k_cache"][0]).copy()
    q = np.ones_like(inputs.bf16_bits_to_f32(att["q"][0]))
    q[:, :, 1::2, :] = -1.0
    for b in range(w.B):
        for lp in range(att["pages_per_seq"]):
            t = lp * 16 + np.arange(16)
            k[att["block_table"][b, lp]] = (level(b, t) / (w.D * att["scale"]))[None, :, None]
    return dict(att, k_cache=[inputs.f32_to_bf16_bits(k)], q=[inputs.f32_to_bf16_bits(q)])


# scores (natural units) by sequence and token: rows that raise their reference once and many times, that leave the range of fp32
# within one stage (the exact pass), whose first scores are far from zero on either side, and whose later ones are
LEVELS = {"slow rise": lambda b, t: np.maximum(t - 150 - 33 * b, 0) * 0.25,
          "one step of 300": lambda b, t: np.where(t > 200 + 41 * b, 300.0, 0.0),
          "two steps of 60": lambda b, t: 60.0 * (t > 170 + 37 * b) + 60.0 * (t > 400),
          "all at 200": lambda b, t: 200.0 + 0.0 * t,
          "down from 150": lambda b, t: np.where(t > 90 + 29 * b, -150.0, 150.0)}


@pytest.mark.parametrize("case", [SHAPES[0], SHAPES[3], SHAPES[4], SHAPES[7], SHAPES[8], SHAPES[9]], ids=lambda c: "tile%d_split%d_K%d" % (c[5], c[6], c[1]))
@pytest.mark.parametrize("level", LEVELS, ids=lambda x: x.replace(" ", "_"))
def test_score_ranges(case, level):
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(14)
    att = scored(w, inputs.make_attention_inputs(w, seed=14), LEVELS[level])
    parent = trees(rng, B, K)
    n_nodes = np.full(B, K, np.int32)
    prefix = (P - rng.integers(0, P // 4, B)).astype(np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1))


@pytest.mark.parametrize("case", [SHAPES[0], SHAPES[6], SHAPES[9]], ids=lambda c: "tile%d_split%d" % c[5:])
def test_tree_slots_far_below_zero(case):
    """No prefix: a workgroup has tree slots only, the first ones hidden from most rows, and scores of -200 that underflow against
    a reference of zero; rows that see nothing of a wavefront's keys are no reason to look again."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(15)
    att = scored(w, inputs.make_attention_inputs(w, seed=15), lambda b, t: -200.0 - 0.125 * t)
    parent = trees(rng, B, K)
    n_nodes = rng.integers(K // 2, K + 1, B).astype(np.int32)
    prefix = (np.arange(B) % 3).astype(np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1))


# every tile, with one split and with several
RANGES = [SHAPES[0], SHAPES[3], SHAPES[4], SHAPES[6], SHAPES[8], SHAPES[9]]


def with_values(att, log2_scale):
    v = inputs.bf16_bits_to_f32(att["v_cache"][0]) * np.float32(2.0 ** log2_scale)        # (exact)
    assert np.abs(v).max() < 2.0 ** 100
    return dict(att, v_cache=[inputs.f32_to_bf16_bits(v)])


def compare_scaled(w, att, parent, n_nodes, prefix, got, rows, log2_scale):
    ref = reference(w, att, parent, n_nodes, prefix, rows)
    assert np.isfinite(got).all()
    err = np.abs(np.stack([got[r] for r in rows]) - ref).max() * 2.0 ** -log2_scale
    print("%d rows, max abs err %.3e of 2^%d" % (len(rows), err, log2_scale))
    assert err <= TOL_BF16


@pytest.mark.parametrize("case", RANGES, ids=lambda c: "tile%d_split%d" % c[5:])
@pytest.mark.parametrize("log2_scale", [-100, 97])
@pytest.mark.parametrize("scores", ["random", "all at -15", "all at 10.9"])
def test_value_magnitudes(case, log2_scale, scores):
    """Values up to the 2^100 that the interface allows and down to the other end, with scores around zero, and, in log2 units, just
    above the bound up to which a reference is zero and as far below."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(22)
    att = with_values(inputs.make_attention_inputs(w, seed=22), log2_scale)
    if scores != "random":
        att = scored(w, att, lambda b, t: float(scores.split()[-1]) + 0.0 * t)
    parent = trees(rng, B, K)
    n_nodes = rng.integers(K // 2, K + 1, B).astype(np.int32)
    prefix = (P - rng.integers(0, P // 4, B)).astype(np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    compare_scaled(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1), log2_scale)


@pytest.mark.parametrize("case", RANGES, ids=lambda c: "tile%d_split%d" % c[5:])
@pytest.mark.parametrize("jump,log2_scale", [(21, 97), (42, 70), (65, 97)])
@pytest.mark.parametrize("last", [32, 64, 0], ids=["last_32", "last_64", "tree"])
def test_last_tokens_far_above_all_others(case, jump, log2_scale, last):
    """Scores that jump in a sequence's last sub-tiles, behind the last look at the sums, under values whose products with them leave
    the range of fp32."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(23)
    n_nodes = rng.integers(K // 2, K + 1, B).astype(np.int32)
    prefix = (P - rng.integers(0, P // 4, B)).astype(np.int32)
    first = prefix + n_nodes - last if last else prefix - 2
    att = scored(w, with_values(inputs.make_attention_inputs(w, seed=23), log2_scale), lambda b, t: np.where(t >= first[b], float(jump), 0.0))
    parent = trees(rng, B, K)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    rows = sample(rng, w, n_nodes, 30 // B + 1) + [(b, int(n_nodes[b]) - 1 - i, 2 * i) for b in range(B) for i in range(3)]
    compare_scaled(w, att, parent, n_nodes, prefix, got, rows, log2_scale)


@pytest.mark.parametrize("case", RANGES, ids=lambda c: "tile%d_split%d" % c[5:])
@pytest.mark.parametrize("level", [-8, -30, -62])
@pytest.mark.parametrize("log2_scale", [-100, 97])
def test_rows_that_see_late_tokens_with_low_scores_only(case, level, log2_scale):
    """No prefix: nodes see a few slots behind a wavefront's first sub-tile, whose scores would be nothing against a
    reference of zero times small values."""
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(24)
    att = scored(w, with_values(inputs.make_attention_inputs(w, seed=24), log2_scale), lambda b, t: level - 0.03125 * t)
    parent = trees(rng, B, K)
    n_nodes, prefix = np.full(B, K, np.int32), (np.arange(B) % 3).astype(np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    rows = sample(rng, w, n_nodes, 30 // B + 1) + [(b, K - 1 - i, 2 * i) for b in range(B) for i in range(4)]
    compare_scaled(w, att, parent, n_nodes, prefix, got, rows, log2_scale)


def test_peaked_softmax():
    w = shape_workload(2, 96, 64, 8, 128, 3000)
    att = inputs.make_attention_inputs(w, seed=12)
    att["q"] = [inputs.f32_to_bf16_bits(inputs.bf16_bits_to_f32(att["q"][0]) * 6.0)]
    rng = np.random.default_rng(12)
    parent = trees(rng, w.B, w.K)
    n_nodes, prefix = np.full(w.B, w.K, np.int32), np.full(w.B, w.P, np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, 3, True)
    rows = sample(rng, w, n_nodes, 60)
    ref = reference(w, att, parent, n_nodes, prefix, rows)
    score_scale_tolerance(np.stack([got[r] for r in rows]), ref, float(np.sqrt(w.D) * att["scale"] * 6.0), "peaked softmax")


@pytest.mark.parametrize("bits", [0x7fc0, 0x7f80, 0xff7f], ids=["nan", "inf", "lowest"])
@pytest.mark.parametrize("case", [SHAPES[0], SHAPES[3], SHAPES[5], SHAPES[9]], ids=lambda c: "tile%d_split%d" % c[5:])
def test_queries_of_absent_nodes_may_hold_anything(case, bits):
    B, K, Hq, Hkv, P, tile, split = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(3)
    att = inputs.make_attention_inputs(w, seed=3)
    n_nodes = rng.integers(K // 3, K, B).astype(np.int32)
    q = att["q"][0].copy()
    for b in range(B):
        q[b, n_nodes[b]:] = bits
    att["q"] = [q]
    parent, prefix = trees(rng, B, K), np.full(B, P, np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, split)
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1))


@pytest.mark.parametrize("B,tile", [(1, 3), (2, 6)])
def test_more_stages_than_a_register_of_pages(B, tile):
    """A wavefront holds the pages of 64 stages; 74 here."""
    w = shape_workload(B, 24, 32, 2, 128, 300000)
    assert attn_plan(B, 24, 32, 2, 128, (300000 + 24 + 15) // 16, "bf16").splits == 64
    rng = np.random.default_rng(6)
    att = inputs.make_attention_inputs(w, seed=6)
    parent = trees(rng, B, 24)
    n_nodes, prefix = np.full(B, 24, np.int32), np.full(B, 300000, np.int32)
    prefix[B - 1] -= 4567
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert_wide(plan, tile, True)
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 4))
