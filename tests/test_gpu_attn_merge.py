"""The kernels that merge an attention call's splits, at the numbers of splits where they take another form: as many as are read at once (2,
4, 8, 12, 16; direct path 8, 16), one more, several wavefronts a row (MI355X only).

Every dim of the result is the weight of its own 1/D of the tokens, so a split that is left out, taken twice or weighed against the wrong
reference changes whole dims by its factor, and rows of the workspace that no split has written hold NaN.  Weights: a token's score is
r in -4 .. 4 (times the node's factor, 1 or 1/2), different from one 1/D to the next, so the splits' references differ.

Relative bound.  bf16: the scaled query is rounded once (2^-9, D = 128, 16-row blocks), so a score is off by 4 * 2^-9 and a weight by twice
that against its row's sum; probabilities are rounded to bf16 (2^-9, in the sum too), results to bf16 (2^-9), partial rows to fp16
(2^-12 of a row's largest dim, so that much of the largest result).  fp32: 21 bits of a score, T sums."""
import numpy as np
import pytest
import torch

import inputs
import paper_2605_20104_amd as graft
from gpu_util import attn_plan, dev, host
from test_gpu_attn import gpu_mask

pytestmark = pytest.mark.gpu

CASES = [  # dtype, D, B, K, Hq, Hkv, P, splits, kernel
    ("bf16", 128, 4, 48, 64, 4, 700, 4, "mfma"), ("bf16", 128, 2, 48, 64, 4, 2600, 5, "mfma"), ("bf16", 128, 2, 48, 64, 4, 4000, 8, "mfma"),
    ("bf16", 128, 3, 50, 8, 2, 1500, 9, "mfma"), ("bf16", 128, 1, 128, 16, 4, 2000, 12, "mfma"), ("bf16", 128, 1, 128, 16, 4, 2300, 13, "mfma"),
    ("bf16", 128, 1, 128, 16, 4, 1800, 16, "mfma"), ("bf16", 128, 2, 33, 16, 2, 4500, 18, "mfma"), ("bf16", 128, 1, 48, 16, 1, 9000, 36, "mfma"),
    ("bf16", 128, 1, 24, 8, 1, 32000, 56, "mfma"),
    ("bf16", 128, 8, 48, 64, 4, 2600, 2, "wide"), ("bf16", 128, 4, 48, 64, 4, 2600, 4, "wide"), ("bf16", 128, 2, 48, 64, 4, 6000, 8, "wide"),
    ("bf16", 128, 1, 48, 64, 4, 12000, 16, "wide"), ("bf16", 128, 1, 96, 32, 2, 16000, 21, "wide"),
    ("bf16", 128, 2, 33, 16, 2, 1800, 3, "direct"), ("bf16", 128, 1, 16, 4, 1, 4500, 9, "direct"), ("bf16", 64, 2, 33, 16, 2, 2600, 3, "direct"),
    ("bf16", 64, 1, 16, 4, 1, 4000, 8, "direct"), ("f32", 64, 1, 16, 4, 1, 1100, 9, "direct"), ("f32", 64, 3, 50, 8, 2, 1500, 4, "parts"),
    ("f32", 128, 1, 16, 4, 1, 4000, 16, "direct"), ("f32", 128, 1, 16, 4, 1, 4500, 18, "direct"), ("f32", 128, 1, 33, 16, 2, 2000, 8, "parts"),
]


@pytest.mark.parametrize("dtype,D,B,K,Hq,Hkv,P,splits,kernel", CASES)
@pytest.mark.parametrize("share", [1.0, 0.4], ids=["full", "short"])
def test_every_split_counts_once(dtype, D, B, K, Hq, Hkv, P, splits, kernel, share):
    rng = np.random.default_rng(P + splits)
    pages = (P + K + 15) // 16
    plan = attn_plan(B, K, Hq, Hkv, D, pages, dtype)
    assert plan.splits == splits and plan.kernel == "tree_attn_%s_kernel" % kernel, plan
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    p = np.array([int(P * share) + 7 * b for b in range(B)], np.int32)       # (short: the last splits have no keys)
    p = np.minimum(p, P)
    n = np.array([K - (b % 3) for b in range(B)], np.int32)
    parent = np.stack([inputs.random_recursive_tree(rng, K, 8) for _ in range(B)])
    table = rng.permutation(B * pages).astype(np.int32).reshape(B, pages)
    k = torch.zeros((B * pages, Hkv, 16, D))
    v = torch.zeros((B * pages, Hkv, 16, D))
    r = rng.integers(-4, 5, (B, Hkv, D)).astype(np.float64)
    own = [np.arange(p[b] + n[b]) * D // (p[b] + n[b]) for b in range(B)]    # a token's dim
    for b in range(B):
        t = np.arange(len(own[b]))
        at = torch.from_numpy(table[b][t // 16].astype(np.int64))
        for g in range(Hkv):
            k[at, g, torch.from_numpy(t % 16), 0] = torch.from_numpy(r[b, g][own[b]]).float()
            v[at, g, torch.from_numpy(t % 16), torch.from_numpy(own[b])] = 1.0
    q = torch.zeros((B, K, Hq, D))
    q[:, 0::2, :, 0], q[:, 1::2, :, 0] = D ** 0.5, 0.5 * D ** 0.5
    q = q.to(kind)
    need = graft.graft_tree_attn_workspace_bytes(B, K, Hq, Hkv, D, pages, graft.GRAFT_F32 if dtype == "f32" else graft.GRAFT_BF16)
    ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")
    out = torch.full((B, K, Hq, D), 7.0, dtype=kind, device="cuda")
    strides = {"page": Hkv * 16 * D, "token": D, "head": 16 * D}
    graft.graft_tree_attn(q.cuda(), k.to(kind).cuda(), v.to(kind).cuda(), strides, dev(table), dev(p), dev(n), gpu_mask(parent, n, p), Hkv, D ** -0.5,
                          out=out, workspace=ws)
    got = host(out).astype(np.float64)
    q0 = q[..., 0].double().numpy()
    if dtype == "f32":
        bound = np.expm1(2 * 4 * 2.0 ** -21) + (P + K) * 2.0 ** -24
    else:
        bound = np.expm1(2 * 4 * 2.0 ** -9) + 3 * 2.0 ** -9
    for b in range(B):
        assert (got[b, n[b]:] == 0).all()
        for i in range(n[b]):
            see = np.zeros(p[b] + n[b], bool)
            see[:p[b]] = True
            j = i
            while j >= 0:
                see[p[b] + j] = True
                j = parent[b, j] if j > 0 else -1
            count = np.bincount(own[b][see], minlength=D)[None]
            for g in range(Hkv):
                h = slice(g * (Hq // Hkv), (g + 1) * (Hq // Hkv))
                w = count * np.exp(r[b, g][None] * q0[b, i, h][:, None] * D ** -0.5)
                ref = w / w.sum(1, keepdims=True)
                slack = 0.0 if dtype == "f32" else ref.max(1, keepdims=True) * 2.0 ** -12
                assert (np.abs(got[b, i, h] - ref) <= bound * ref + slack).all(), (b, i, g, np.abs(got[b, i, h] - ref).max())
