"""GPU parity of the MFMA attention kernel (bf16, D = 128) against the CPU oracle, in shapes for which the library takes
that path: every test asserts it, and where the kernel has variants, which one (MI355X only).

Tolerance as for every bf16 test with D = 128: 2e-2 (test_gpu_attn.py says where it comes from)."""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2605_20104_amd as graft
from gpu_util import attn_plan, dev, host, widened
from test_gpu_attn import TOL_BF16, gpu_mask, score_scale_tolerance, shape_workload

pytestmark = pytest.mark.gpu


def run(w, att, parent, n_nodes, prefix):
    """Output [B,K,Hq,D] and the plan; asserts the path."""
    plan = attn_plan(w.B, w.K, w.Hq, w.Hkv, w.D, att["block_table"].shape[1], w.dtype)
    assert plan.path == "mfma", plan
    mask = gpu_mask(parent, n_nodes, prefix)
    out = torch.full((w.B, w.K, w.Hq, w.D), 7.0, dtype=torch.bfloat16, device="cuda")
    graft.graft_tree_attn(dev(att["q"][0], "bf16"), dev(att["k_cache"][0], "bf16"), dev(att["v_cache"][0], "bf16"), att["strides"],
                          dev(att["block_table"]), dev(prefix), dev(n_nodes), mask, w.Hkv, att["scale"], out=out)
    return host(out).astype(np.float64), plan


def main_kernel(row_blocks):
    """Tiles of 256 rows have the kernel with 32-row blocks only; those of 192 here have too few stages for it."""
    return "tree_attn_wide_kernel" if row_blocks == 4 else "tree_attn_mfma_kernel"


def reference(w, att, parent, n_nodes, prefix, rows=None):
    return oracle.tree_attn(att["q"][0], att["k_cache"][0], att["v_cache"][0], "bf16", att["strides"], att["block_table"], prefix,
                            n_nodes, parent, w.Hq, w.Hkv, w.D, w.page_size, att["scale"], rows=rows)


def sample(rng, w, n_nodes, per_sequence):
    """Rows (sequence, node, head): the first and the last live one of every sequence and some between."""
    rows = [(b, int(rng.integers(n)), int(rng.integers(w.Hq))) for b, n in enumerate(n_nodes) if n for _ in range(per_sequence)]
    return rows + [(b, i, h) for b, n in enumerate(n_nodes) if n for i, h in ((0, 0), (n - 1, w.Hq - 1))]


def compare(w, att, parent, n_nodes, prefix, got, rows):
    ref = reference(w, att, parent, n_nodes, prefix, rows)
    assert np.isfinite(got).all()
    err = np.abs(np.stack([got[r] for r in rows]) - ref)
    print("%d rows, max abs err %.3e" % (len(rows), err.max()))
    assert err.max() <= TOL_BF16
    for b, n in enumerate(n_nodes):
        assert (got[b, n:] == 0).all()


# (B, K, Hq, Hkv, P, row blocks): a natural table, at least three 64-token stages per workgroup
NATURAL = [(1, 128, 2, 1, 3000, 1), (8, 16, 32, 8, 4000, 1), (1, 80, 20, 4, 2000, 2), (8, 65, 32, 4, 200, 2), (4, 128, 40, 8, 200, 3),
           (2, 65, 16, 1, 3000, 3), (8, 65, 32, 2, 500, 4), (1, 80, 128, 8, 1000, 4), (8, 65, 128, 8, 200, 5), (8, 80, 64, 8, 500, 5)]


@pytest.mark.parametrize("case", NATURAL, ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_mb%d" % c)
@pytest.mark.parametrize("layout", ["head_major", "token_major"])
def test_every_number_of_row_blocks(case, layout):
    """Ragged prefixes and trees (lengths off every boundary of 16, 32 and 64), trees across both 64-bit mask words and
    across 32-bit words, both cache layouts."""
    B, K, Hq, Hkv, P, mb = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(P + K)
    att = inputs.make_attention_inputs(w, seed=P + K, layout=layout)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8 if b % 2 else K - 1) for b in range(B)])
    n_nodes, prefix = np.full(B, K, np.int32), np.full(B, P, np.int32)
    n_nodes[1:], prefix[1:] = rng.integers(1, K + 1, B - 1), rng.integers(P // 2, P + 1, B - 1)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert (plan.row_blocks, plan.kernel) == (mb, main_kernel(mb)), plan
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 60 // B + 1))


# (B, K, Hq, Hkv, P, pages): short sequences in a table long enough for this path: most splits have nothing to do
SHORT = [(1, 1, 1, 1, 0, 1), (1, 1, 8, 8, 5, 1), (2, 16, 8, 2, 333, 133), (1, 40, 32, 8, 1000, 97), (1, 64, 40, 8, 777, 145), (2, 48, 32, 2, 300, 145),
         (1, 96, 8, 2, 1201, 321), (1, 128, 4, 2, 130, 97), (3, 33, 6, 2, 64, 97), (1, 20, 16, 16, 31, 4), (1, 128, 32, 2, 100, 225)]


@pytest.mark.parametrize("case", SHORT, ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_pages%d" % c)
def test_short_sequences(case):
    B, K, Hq, Hkv, P, pages = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(K + P)
    att = widened(inputs.make_attention_inputs(w, seed=K + P), pages)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    n_nodes, prefix = np.full(B, K, np.int32), np.full(B, P, np.int32)
    got, _ = run(w, att, parent, n_nodes, prefix)
    compare(w, att, parent, n_nodes, prefix, got, [(b, i, h) for b in range(B) for i in range(K) for h in range(Hq)])


def test_ragged_batch_padding_nodes_and_an_invalid_tree():
    w = shape_workload(4, 48, 16, 4, 128, 500)
    att = widened(inputs.make_attention_inputs(w, seed=5), 145)
    rng = np.random.default_rng(5)
    parent = np.stack([inputs.random_recursive_tree(rng, w.K, 8) for _ in range(w.B)])
    n_nodes, prefix = np.array([48, 1, 33, 0], np.int32), np.array([17, 0, 123, 500], np.int32)
    got, _ = run(w, att, parent, n_nodes, prefix)
    compare(w, att, parent, n_nodes, prefix, got, [(b, i, h) for b in range(w.B) for i in range(n_nodes[b]) for h in range(w.Hq)])


def test_token_major_layout_and_deep_chain():
    w = shape_workload(2, 64, 8, 2, 128, 200)
    att = widened(inputs.make_attention_inputs(w, seed=6, layout="token_major"), 81)
    rng = np.random.default_rng(6)
    parent = np.stack([inputs.random_recursive_tree(rng, w.K, 63), np.arange(-1, w.K - 1)]).astype(np.int32)
    n_nodes, prefix = np.full(2, w.K, np.int32), np.full(2, w.P, np.int32)
    got, _ = run(w, att, parent, n_nodes, prefix)
    compare(w, att, parent, n_nodes, prefix, got, [(b, i, h) for b in range(2) for i in range(w.K) for h in range(w.Hq)])


def test_large_scores_stay_finite():
    """Peaked softmax (large |q.k|): the lazy running max must not overflow."""
    w = shape_workload(1, 16, 8, 2, 128, 400)
    att = widened(inputs.make_attention_inputs(w, seed=12), 133)
    att["q"] = [inputs.f32_to_bf16_bits(inputs.bf16_bits_to_f32(att["q"][0]) * 6.0)]
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(12), w.K, 8)])
    n_nodes, prefix = np.array([w.K], np.int32), np.array([w.P], np.int32)
    got, _ = run(w, att, parent, n_nodes, prefix)
    assert np.isfinite(got).all()
    score_scale_tolerance(got, reference(w, att, parent, n_nodes, prefix), float(np.sqrt(w.D) * att["scale"] * 6.0), "peaked softmax")


# (B, K, Hq, Hkv, P, row blocks, rise per token in units of the keys)
RISING = [(8, 16, 32, 8, 4000, 1, 0.0153), (1, 128, 2, 1, 3000, 1, 0.0153), (8, 24, 32, 8, 1500, 2, 0.0153), (2, 65, 16, 1, 3000, 3, 0.0153),
          (8, 65, 32, 2, 500, 4, 0.03), (8, 80, 64, 8, 500, 5, 0.03)]


@pytest.mark.parametrize("case", RISING, ids=lambda c: "B%d_K%d_Hq%d_Hkv%d_P%d_mb%d_rise%g" % c)
def test_scores_that_outgrow_the_reference(case):
    """Scores that are flat for a while and then rise by far more than the lazy bound of the fast loop, from another place in
    every sequence, so that wavefronts leave it at even and at odd sub-tiles with transfers of later stages still to be issued
    (exact running maximum from there on); falling scores stay in it."""
    B, K, Hq, Hkv, P, mb, rise = case
    w = shape_workload(B, K, Hq, Hkv, 128, P)
    rng = np.random.default_rng(14)
    att = inputs.make_attention_inputs(w, seed=14)
    k = inputs.bf16_bits_to_f32(att["k_cache"][0]).copy()
    q = np.ones_like(inputs.bf16_bits_to_f32(att["q"][0]))
    q[:, :, 1::2, :] = -1.0                                                  # odd heads: falling scores
    prefix = (P - rng.integers(0, P // 4, B)).astype(np.int32)
    for b in range(B):
        for lp in range(att["pages_per_seq"]):
            t = lp * 16 + np.arange(16)
            k[att["block_table"][b, lp]] = (np.maximum(t - (50 + 33 * b), 0) * rise)[None, :, None]
    att["k_cache"], att["q"] = [inputs.f32_to_bf16_bits(k)], [inputs.f32_to_bf16_bits(q)]
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    n_nodes = np.full(B, K, np.int32)
    got, plan = run(w, att, parent, n_nodes, prefix)
    assert (plan.row_blocks, plan.kernel) == (mb, main_kernel(mb)), plan
    assert rise * (P // 2) * w.D * att["scale"] * 1.44 > 2 * 24              # twice the lazy bound in log2 units
    compare(w, att, parent, n_nodes, prefix, got, sample(rng, w, n_nodes, 80 // B + 1))


@pytest.mark.parametrize("P,pages", [(450, 133), (2100, 133)])
def test_agrees_with_the_direct_kernel(P, pages):
    """The two GPU paths on the same inputs, which share no tiling, masking or merging code beyond the mask window: bf16
    through the MFMA kernel and, widened to fp32, through the direct one."""
    w = shape_workload(1, 24, 8, 2, 128, P)
    att = widened(inputs.make_attention_inputs(w, seed=11), pages)
    parent = np.stack([inputs.random_recursive_tree(np.random.default_rng(11), w.K, 8)])
    n_nodes, prefix = np.array([w.K], np.int32), np.array([w.P], np.int32)
    got, _ = run(w, att, parent, n_nodes, prefix)
    assert attn_plan(w.B, w.K, w.Hq, w.Hkv, w.D, pages, "f32").path == "direct"
    f32 = lambda a: dev(inputs.bf16_bits_to_f32(a), "f32")
    direct = host(graft.graft_tree_attn(f32(att["q"][0]), f32(att["k_cache"][0]), f32(att["v_cache"][0]), att["strides"], dev(att["block_table"]),
                                        dev(prefix), dev(n_nodes), gpu_mask(parent, n_nodes, prefix), w.Hkv, att["scale"])).astype(np.float64)
    assert np.abs(direct - reference(w, att, parent, n_nodes, prefix)).max() <= 1e-4
    assert np.abs(direct - got).max() <= TOL_BF16
