"""Helpers for the GPU parity tests: host<->device transfers and workload runners."""
import collections
import ctypes

import numpy as np
import torch

import paper_2605_20104_amd as graft
from paper_2605_20104_amd import build


def dev(a, dtype="i32"):
    """numpy -> cuda tensor.  dtype 'bf16' takes uint16 storage bits."""
    if a is None:
        return None
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).cuda()
    if dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def host(t):
    """cuda tensor -> numpy; bfloat16 comes back widened to float32; mask words as uint64."""
    if t is None:
        return None
    if t.dtype == torch.bfloat16:
        return t.float().cpu().numpy()
    if t.dtype == torch.int64:
        return t.cpu().numpy().view(np.uint64)
    return t.cpu().numpy()


def host_dict(d):
    torch.cuda.synchronize()
    return {k: host(v) for k, v in d.items()}


def assert_same(gpu: dict, ref: dict, keys):
    for k in keys:
        a, b = gpu[k], ref[k]
        assert a.shape == b.shape, (k, a.shape, b.shape)
        assert (a == b).all(), "%s differs:\n gpu %s\n ref %s" % (k, a.ravel()[:32], b.ravel()[:32])


def run_attn(att, dtype, prefix_len, n_nodes, mask, Hkv, layer=0, kv=0):
    """att: dict from inputs.make_attention_inputs (or same keys).  Returns float32 numpy [B,K,Hq,D]."""
    q = dev(att["q"][layer], dtype)
    k = dev(att["k_cache"][kv], dtype)
    v = dev(att["v_cache"][kv], dtype)
    out = graft.graft_tree_attn(q, k, v, att["strides"], dev(att["block_table"]), dev(prefix_len),
                                dev(n_nodes), mask, Hkv, att["scale"])
    torch.cuda.synchronize()
    return host(out).astype(np.float32)


def us_per_call(call, reps=20):
    """Duration of `call(stream)` on the GPU: the median of seven replays of a graph of `reps` calls."""
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        call(side)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(reps):
            call(torch.cuda.current_stream())
    times = []
    graph.replay()
    for _ in range(7):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        graph.replay()
        stop.record()
        stop.synchronize()
        times.append(start.elapsed_time(stop) * 1000 / reps)
    return sorted(times)[3]


AttnPlan = collections.namedtuple("AttnPlan", "path row_blocks row_tiles splits kernel")


def attn_plan(B, K, Hq, Hkv, D, max_pages, dtype):
    """The path ("mfma" or "direct"), launch shape and main kernel of an attention call, as the timing build tells it: the
    product library plans with the same code."""
    lib = ctypes.CDLL(build.LIB_TIMING)
    lib.graft_attn_kernel_name.restype = ctypes.c_char_p
    shape = (B, K, Hq, Hkv, D, max_pages, graft.GRAFT_F32 if dtype == "f32" else graft.GRAFT_BF16)
    plan = (ctypes.c_int32 * 4)()
    assert lib.graft_attn_plan(*shape, plan) == 0
    return AttnPlan(("direct", "mfma")[plan[0]], *plan[1:], lib.graft_attn_kernel_name(*shape).decode())


def widened(att, pages):
    """The same inputs with a block table of more pages (the launch is planned from its capacity); what is added is not used."""
    table = att["block_table"]
    wide = np.zeros((table.shape[0], pages), np.int32)
    wide[:, :table.shape[1]] = table
    return dict(att, block_table=wide)
