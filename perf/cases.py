"""Work that users of this package have it do, as cases whose time can be measured.

Five kinds of work, each through the package's public calls:

  round     the verification round of one decoding step: graft_retrieve, graft_build_tree_mask,
            graft_tree_attn once per layer, graft_accept.  A serving loop keeps its output buffers
            and workspaces, so these are handed in.
  retrieve  graft_retrieve alone, over a context buffer that has grown long.
  prepare   draft tree to hybrid tree: graft_prune_select, graft_matrix_retrieve (which appends to
            the tree that pruning returned), graft_build_tree_mask; outputs allocated by the calls.
  refresh   what follows the target model: graft_matrix_update over the logits, graft_accept with
            the ids it returns, graft_kv_compact over all layers.  layers = 0 is the refresh from a
            prefill, where the prompt's positions are handed over as rows and nothing is accepted.
  accept    graft_accept over the target's logits.

A case fixes the sizes; prepare() draws the values from the seed: Zipf-distributed contexts with a
planted query n-gram, random draft trees with grafted chains, N(0,1) queries, keys, values and
logits, random page tables.
"""
import math

import numpy as np
import torch

import paper_2605_20104_amd as graft

PAGE = graft.GRAFT_PAGE_SIZE
DEPTH_CAP = 48


def listed():
    rnd = dict(kind="round", dtype="bf16", D=128, layout="head_major", ragged=False, n_min=2, n_max=8, C=3, m=8)
    return [
        # The smallest: one layer of a toy model in fp32, 16 tree nodes over 256 tokens.  Latency,
        # launches and host time are all there is.
        dict(rnd, name="round_tiny_f32", dtype="f32", B=1, layers=1, Hq=8, Hkv=2, D=64, P=256, K=16, L=256, V=1000,
             n_min=4, n_max=4, C=1, m=4),
        # One chat request on an 8B-class model: 32 layers, a 2K prefix, 40 tree nodes.
        dict(rnd, name="round_short_32_layers", B=1, layers=32, Hq=32, Hkv=8, P=2048, K=40, L=2048, V=128256, C=2),
        # One request with a 32K prefix (meeting transcripts, repositories), 40 query and 8 KV heads.
        dict(rnd, name="round_long_prefix", B=1, layers=1, Hq=40, Hkv=8, P=32768, K=64, L=32768, V=151936),
        # A serving batch of 8 on one GPU's share of a large model's heads, all 94 layers.
        dict(rnd, name="round_batch_94_layers", B=8, layers=94, Hq=64, Hkv=4, P=4096, K=48, L=4096, V=151936),
        # Four requests with 64K prefixes and a 96-node tree.
        dict(rnd, name="round_long_prefix_batch", B=4, layers=1, Hq=32, Hkv=8, P=65536, K=96, L=65536, V=128256, C=2),
        # A model with head size 64 and the other cache layout, batch of 4 with ragged lengths.
        dict(rnd, name="round_head_64_ragged", B=4, layers=16, Hq=32, Hkv=8, D=64, P=2048, K=60, L=2048, V=128256,
             layout="token_major", ragged=True),
        # fp32 storage and arithmetic (validating a model against its fp32 reference): 8 layers.
        dict(rnd, name="round_f32_8_layers", dtype="f32", B=1, layers=8, Hq=32, Hkv=8, P=2048, K=40, L=2048, V=128256),
        # Acceptance straight from the target's logits, batch of 8.
        dict(name="accept_logits_batch", kind="accept", B=8, K=48, V=151936),
        # After one request's verification: matrix refresh, acceptance, cache update of 32 layers.
        dict(name="refresh_one_request", kind="refresh", B=1, K=40, V=128256, k=8, layers=32, Hkv=8, D=128, P=2048, dtype="bf16"),
        # Matrix refresh from a prefill of 2048 positions.
        dict(name="refresh_prefill", kind="refresh", B=16, K=128, V=128256, k=8, layers=0, Hkv=8, D=128, P=0, dtype="bf16"),
        # Suffix lookup in one request's context of 128K tokens.
        dict(name="retrieve_long_context", kind="retrieve", B=1, L=131072, V=151936, n_min=2, n_max=8, C=3, m=8),
        # Gates, template lookup and masks for a batch of 4 with a budget of 60 nodes.
        dict(name="prepare_tree", kind="prepare", B=4, K=64, budget=60, V=151936, k=8),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["round"] * 5 + ["retrieve", "prepare", "refresh", "accept"])
    B = _log_int(rng, 1, 16)
    V = _log_int(rng, 8000, 152000)
    if kind == "retrieve":
        n_max = rng.randint(3, 16)
        return dict(kind=kind, B=B, L=_log_int(rng, 256, 200000), V=V, n_min=rng.randint(1, 3), n_max=n_max,
                    C=rng.randint(1, 8), m=rng.randint(4, 16))
    if kind == "prepare":
        budget = rng.randint(24, 120)
        return dict(kind=kind, B=B, K=min(128, budget + rng.randint(0, 8)), budget=budget, V=V, k=rng.randint(4, 16))
    if kind == "accept":
        return dict(kind=kind, B=B, K=rng.randint(8, 128 if B <= 8 else 64), V=V)
    if kind == "refresh":
        if rng.random() < 0.3:
            return dict(kind=kind, B=B, K=128, V=V, k=rng.randint(4, 16), layers=0, Hkv=8, D=128, P=0, dtype="bf16")
        return dict(kind=kind, B=B, K=rng.randint(8, 96), V=V, k=rng.randint(4, 16), layers=_log_int(rng, 1, 48),
                    Hkv=rng.choice([1, 2, 4, 8]), D=rng.choice([64, 128]), P=_log_int(rng, 64, 4096),
                    dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
    dtype = rng.choice(["bf16"] * 4 + ["f32"])
    D = rng.choice([128, 128, 128, 64])
    Hkv = rng.choice([1, 2, 4, 8])
    c = dict(kind=kind, dtype=dtype, B=B, layers=1, Hq=Hkv * rng.randint(1, 16), Hkv=Hkv, D=D,
             P=_log_int(rng, 32, 65536), K=rng.randint(8, 128), L=0, V=V, n_min=rng.randint(1, 3), n_max=rng.randint(4, 12),
             C=rng.randint(1, 4), m=rng.randint(4, 12), layout=rng.choice(["head_major", "head_major", "token_major"]),
             ragged=rng.random() < 0.5)
    c["L"] = max(c["P"], 256)
    # as many layers as a model has, as far as the pass stays below the largest listed one
    most = 2e12 if dtype == "bf16" and D == 128 else 6e10
    want = _log_int(rng, 1, 64)
    while work(c)["flops"] > most:
        c["P"] = max(32, c["P"] // 2)
        c["L"] = max(c["P"], 256)
        if c["P"] == 32:
            c["B"] = max(1, c["B"] // 2)
    one = work(c)
    c["layers"] = max(1, min(want, int(most / one["flops"]), int(6e9 / one["bytes"])))
    return c


# ---------------------------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------------------------
def _lengths(c):
    """(prefix length, tree nodes) per sequence; a ragged batch has lengths down to about half."""
    out = []
    for b in range(c["B"]):
        if c.get("ragged"):
            out.append((c["P"] - (b * 997) % (c["P"] // 2 + 1), c["K"] - (b * 7) % (c["K"] // 2 + 1)))
        else:
            out.append((c["P"], c["K"]))
    return out


def work(c):
    kind, B = c["kind"], c["B"]
    if kind == "retrieve":
        return {"bytes": 4.0 * B * (c["L"] + c["C"] * (c["m"] + 3) + 4), "flops": 0.0}
    if kind == "prepare":
        # tree in (3 arrays), kept tree out (3), appended nodes and their lookups, masks and positions out
        return {"bytes": B * (c["K"] * (6 * 4 + 16 + 2 * 4) + c["budget"] * 12 + c["K"] * (DEPTH_CAP + 1) * 4.0), "flops": 0.0}
    if kind == "accept":
        return {"bytes": 4.0 * B * (c["K"] * (c["V"] + 3) + 2 * DEPTH_CAP), "flops": 0.0}
    if kind == "refresh":
        moved = 4 * 2 * 2 * c["layers"] * c["Hkv"] * c["D"] * (2 if c["dtype"] == "bf16" else 4)   # about 4 rows a sequence
        return {"bytes": B * (4.0 * c["K"] * (c["V"] + c["k"] + 2) + moved), "flops": 0.0}
    e = 2 if c["dtype"] == "bf16" else 4
    nbytes, flops = 4.0 * B * c["L"] + B * c["K"] * (16 + 5 * 4 + 4 * (DEPTH_CAP + 1)), 0.0
    for P, n in _lengths(c):
        kv = 2 * (P + n) * c["Hkv"] * c["D"] * e
        qo = (n + c["K"]) * c["Hq"] * c["D"] * e
        nbytes += c["layers"] * (kv + qo + 4 * ((P + n + PAGE - 1) // PAGE) + 16 * n)
        flops += c["layers"] * 4.0 * n * c["Hq"] * c["D"] * (P + min(n, 8))       # the prefix and about 8 nodes of the own path
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(c):
    if c["kind"] != "round":
        return "exact"                     # whole numbers, and cache rows that are moved as they are
    return {"rel": 1e-2 if c["dtype"] == "bf16" else 1e-5, "differ": 0.0}


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _up(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _gpu_rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _tree(rng, n, K, chain, max_depth=6):
    """Parents of n nodes in K slots: a random draft tree, then chains of `chain` nodes appended."""
    parent = np.full(K, -1, np.int32)
    depth = np.zeros(K, np.int32)
    n_draft = n if n < 3 * chain + 4 else n - chain * int(rng.integers(1, 3))
    for i in range(1, n):
        if i < n_draft:
            p = int(rng.integers(max(0, i - 12), i))
            while depth[p] >= max_depth:
                p = int(parent[p])
        else:
            p = int(rng.integers(0, n_draft)) if (i - n_draft) % chain == 0 else i - 1
        parent[i], depth[i] = p, depth[p] + 1
    return parent


def _targets(rng, parent, tokens, n, V):
    """A greedy token per node: a child's token three times out of four, else any."""
    ids = rng.integers(0, V, len(parent)).astype(np.int32)
    for i in range(n - 1, 0, -1):
        if rng.random() < 0.75:
            ids[parent[i]] = tokens[i]
    ids[n:] = -1
    return ids


def _trees(rng, c, lengths, chain=8):
    B, K, V = c["B"], c["K"], c["V"]
    parent = np.stack([_tree(rng, n, K, chain) for _, n in lengths])
    tokens = rng.integers(0, V, (B, K)).astype(np.int32)
    ids = np.stack([_targets(rng, parent[b], tokens[b], lengths[b][1], V) for b in range(B)])
    return parent, tokens, ids


def _contexts(rng, c):
    """Zipf-distributed tokens, the query n-gram (last tokens of context and tail) planted C + 2 times."""
    B, L, V = c["B"], c["L"], c["V"]
    cdf = np.cumsum(1.0 / np.arange(1, V + 1) ** 1.1)
    ids = rng.permutation(V).astype(np.int32)
    ctx = ids[np.minimum(np.searchsorted(cdf, rng.random((B, L)) * cdf[-1]), V - 1)]
    ctx[:, L - c["n_max"]:] = rng.integers(0, V, (B, c["n_max"]))
    tail = rng.integers(0, V, (B, 4)).astype(np.int32)
    tail_len = rng.integers(0, 5, B).astype(np.int32)
    for b in range(B):
        q = np.concatenate([ctx[b], tail[b, :tail_len[b]]])[-c["n_max"]:]
        for _ in range(c["C"] + 2):
            at = int(rng.integers(0, L - 2 * c["n_max"] - c["m"]))
            ctx[b, at:at + len(q)] = q
    return _up(ctx), _up(np.full(B, L)), _up(tail), _up(tail_len)


def _logits(gen, ids, V):
    """N(0,1) rows whose first maximum is the row's greedy token."""
    B, K = ids.shape
    logits = torch.randn((B, K, V), generator=gen, device="cuda")
    at = torch.from_numpy(np.maximum(ids, 0).astype(np.int64)).cuda()[..., None]
    return logits.scatter_(2, at, torch.rand((B, K, 1), generator=gen, device="cuda") + 12.0)


def _caches(gen, c, pages):
    """K and V caches of all layers in one allocation each, and their strides."""
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    Hkv, D = c["Hkv"], c["D"]
    if c.get("layout") == "token_major":
        shape, strides = (PAGE, Hkv, D), {"page": PAGE * Hkv * D, "token": Hkv * D, "head": D}
    else:
        shape, strides = (Hkv, PAGE, D), {"page": PAGE * Hkv * D, "token": D, "head": PAGE * D}
    k, v = (torch.randn((c["layers"], pages) + shape, generator=gen, device="cuda", dtype=dt) for _ in range(2))
    return k, v, strides


def _table(gen, B, per_seq):
    """A pool a quarter larger than what is in use, its pages handed out in random order."""
    pool = B * per_seq + (B * per_seq + 3) // 4
    perm = torch.randperm(pool, generator=gen, device="cuda")
    return perm[:B * per_seq].to(torch.int32).reshape(B, per_seq).contiguous(), pool


def _ints(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def prepare(case, seed):
    return {"round": _prepare_round, "retrieve": _prepare_retrieve, "prepare": _prepare_tree,
            "refresh": _prepare_refresh, "accept": _prepare_accept}[case["kind"]](case, seed)


def _prepare_round(c, seed):
    rng, gen = np.random.default_rng(seed), _gpu_rng(seed)
    B, K, Hq, D = c["B"], c["K"], c["Hq"], c["D"]
    lengths = _lengths(c)
    parent, tokens, ids = _trees(rng, c, lengths, c["m"])
    ctx, ctx_len, tail, tail_len = _contexts(rng, c)
    table, pool = _table(gen, B, (c["P"] + K + PAGE - 1) // PAGE)
    kc, vc, strides = _caches(gen, c, pool)
    q = torch.randn((c["layers"], B, K, Hq, D), generator=gen, device="cuda", dtype=kc.dtype)
    out = torch.zeros_like(q)
    need = graft.graft_tree_attn_workspace_bytes(B, K, Hq, c["Hkv"], D, table.shape[1],
                                                 graft.GRAFT_BF16 if c["dtype"] == "bf16" else graft.GRAFT_F32)
    return dict(
        c=c, ctx=ctx, ctx_len=ctx_len, tail=tail, tail_len=tail_len, parent=_up(parent), tokens=_up(tokens), ids=_up(ids),
        n_nodes=_up([n for _, n in lengths]), prefix_len=_up([P for P, _ in lengths]), table=table, strides=strides,
        layers=[(q[i], kc[i], vc[i], out[i]) for i in range(c["layers"])], out=out, scale=1.0 / math.sqrt(D),
        ws=torch.empty(max(need, 256), dtype=torch.uint8, device="cuda"),
        ret=dict(chain_tok=_ints(B, c["C"], c["m"]), chain_len=_ints(B, c["C"]), chain_pos=_ints(B, c["C"]),
                 chain_match=_ints(B, c["C"]), n_hits=_ints(B), status=_ints(B)),
        mask=dict(mask=torch.empty((B, K, graft.GRAFT_MASK_WORDS), dtype=torch.int64, device="cuda"), pos=_ints(B, K),
                  depth=_ints(B, K), paths=_ints(B, K, DEPTH_CAP + 1), status=_ints(B)),
        acc=dict(accept_len=_ints(B), best_node=_ints(B), path=_ints(B, DEPTH_CAP + 1), out_tokens=_ints(B, DEPTH_CAP + 1),
                 status=_ints(B)))


def _prepare_retrieve(c, seed):
    ctx, ctx_len, tail, tail_len = _contexts(np.random.default_rng(seed), c)
    return dict(c=c, ctx=ctx, ctx_len=ctx_len, tail=tail, tail_len=tail_len)


def _prepare_tree(c, seed):
    rng, gen = np.random.default_rng(seed), _gpu_rng(seed)
    B, K, budget, V, k = c["B"], c["K"], c["budget"], c["V"], c["k"]
    parent, tokens, _ = _trees(rng, c, [(0, budget)] * B, chain=budget)
    logq = np.log(rng.uniform(0.2, 0.95, (B, K))).astype(np.float32)
    keep = np.maximum(1, np.array([8, 24, 40]) * budget // 60)
    n_tpl = min(80, budget)
    tpl_parent, tpl_rank, depth = np.full(n_tpl, -1, np.int32), np.zeros(n_tpl, np.int32), np.ones(n_tpl, np.int32)
    children = np.zeros(n_tpl + 1, np.int32)                    # the last entry counts the root's
    for u in range(n_tpl):
        p = -1 if u < 4 else int(rng.integers(-1, u))
        while children[p] >= min(k, 8) or (p >= 0 and depth[p] >= 9):
            p = int(rng.integers(0, u))
        tpl_parent[u], tpl_rank[u], depth[u] = p, children[p], 1 if p < 0 else depth[p] + 1
        children[p] += 1
    M = torch.randint(-1, V, (V, k), generator=gen, device="cuda", dtype=torch.int32)
    return dict(c=c, parent=_up(parent), tokens=_up(tokens), logq=torch.from_numpy(logq).cuda(),
                n_nodes=_up([budget] * B), prefix_len=_up(rng.integers(100, 5000, B)), M=M,
                chk_depth=_up([1, 2, 6]), chk_log_tau=torch.tensor([-0.5, -1.5, -3.0], device="cuda"), chk_keep=_up(keep),
                chk_ret=_up(np.minimum(n_tpl, budget - keep)), tpl_parent=_up(tpl_parent), tpl_rank=_up(tpl_rank))


def _prepare_refresh(c, seed):
    rng, gen = np.random.default_rng(seed), _gpu_rng(seed)
    B, K = c["B"], c["K"]
    parent, tokens, ids = _trees(rng, c, [(c["P"], K)] * B)
    s = dict(c=c, parent=_up(parent), tokens=_up(tokens), n_nodes=_up([K] * B), logits=_logits(gen, ids, c["V"]),
             M=torch.full((c["V"], c["k"]), -1, dtype=torch.int32, device="cuda"))
    if c["layers"]:
        s["table"], pool = _table(gen, B, (c["P"] + K + PAGE - 1) // PAGE)
        s["kc"], s["vc"], s["strides"] = _caches(gen, c, pool)
        s["prefix_len"] = _up([c["P"]] * B)
    return s


def _prepare_accept(c, seed):
    rng, gen = np.random.default_rng(seed), _gpu_rng(seed)
    parent, tokens, ids = _trees(rng, c, [(0, c["K"])] * c["B"])
    return dict(c=c, parent=_up(parent), tokens=_up(tokens), n_nodes=_up([c["K"]] * c["B"]), logits=_logits(gen, ids, c["V"]))


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "retrieve":
        return graft.graft_retrieve(s["ctx"], s["ctx_len"], c["n_min"], c["n_max"], c["C"], c["m"], s["tail"], s["tail_len"])
    if kind == "accept":
        return graft.graft_accept(s["parent"], s["tokens"], s["n_nodes"], DEPTH_CAP, logits=s["logits"])
    if kind == "prepare":
        t = graft.graft_prune_select(s["parent"], s["tokens"], s["logq"], s["n_nodes"], s["chk_depth"], s["chk_log_tau"],
                                     s["chk_keep"], s["chk_ret"])
        status = graft.graft_matrix_retrieve(s["M"], s["tpl_parent"], s["tpl_rank"], t["n_ret"], t["tokens"], t["parent"],
                                             t["n_nodes"])
        mask = graft.graft_build_tree_mask(t["parent"], t["n_nodes"], s["prefix_len"], c["K"], DEPTH_CAP)
        return {"tree": t, "status": status, "mask": mask}
    if kind == "refresh":
        ids = graft.graft_matrix_update(s["tokens"], s["n_nodes"], s["logits"], s["M"])
        if not c["layers"]:
            return {"M": s["M"], "target_ids": ids}
        acc = graft.graft_accept(s["parent"], s["tokens"], s["n_nodes"], DEPTH_CAP, target_ids=ids)
        moved = graft.graft_kv_compact(s["kc"], s["vc"], s["kc"].stride(0), c["layers"], s["strides"], s["table"],
                                       s["prefix_len"], acc["path"], acc["accept_len"], c["K"], c["Hkv"], c["D"])
        return {"M": s["M"], "accept": acc, "k_cache": s["kc"], "v_cache": s["vc"], "moved": moved}
    ret = graft.graft_retrieve(s["ctx"], s["ctx_len"], c["n_min"], c["n_max"], c["C"], c["m"], s["tail"], s["tail_len"],
                               out=s["ret"])
    mask = graft.graft_build_tree_mask(s["parent"], s["n_nodes"], s["prefix_len"], c["K"], DEPTH_CAP, out=s["mask"])
    for q, k, v, out in s["layers"]:
        graft.graft_tree_attn(q, k, v, s["strides"], s["table"], s["prefix_len"], s["n_nodes"], mask["mask"], c["Hkv"],
                              s["scale"], out=out, workspace=s["ws"])
    acc = graft.graft_accept(s["parent"], s["tokens"], s["n_nodes"], DEPTH_CAP, target_ids=s["ids"], out=s["acc"])
    return {"chains": ret, "mask": mask, "attention": s["out"], "accept": acc}
