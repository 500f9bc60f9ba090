"""Thin Python binding of libgraft.so, the C-ABI library declared in include/graft.h.

Argument marshalling only: every step of the verification path runs in the HIP
kernels behind the entry points.  PyTorch is used for device memory and streams; tensors are
passed as raw device pointers.  The marshalling itself is native (csrc/binding.cpp, built as
_native.so next to the library).  A workspace that a call has to allocate belongs to the stream
the call runs on (`stream`, by default the current one); results that it allocates belong to
the current stream, as every tensor does, so with another `stream` they are kept until it is done.  There is no CPU fallback: if the library is not built the
first call raises.
"""
from __future__ import annotations

import ctypes
import os

import torch  # noqa: F401  (device memory and streams; its libraries must be loaded before the native module)

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libgraft.so")
NATIVE_PATH = os.path.join(_PKG, "_native.so")

GRAFT_MAX_NODES = 128
GRAFT_MASK_WORDS = 2
GRAFT_MAX_CHAINS = 8
GRAFT_MAX_NGRAM = 32
GRAFT_PAGE_SIZE = 16
GRAFT_MAX_SUCCESSORS = 16
GRAFT_MAX_CHECKPOINTS = 16
GRAFT_NOALLOC_MAX_ROWS = 8192
GRAFT_OK, GRAFT_ERR_NULL, GRAFT_ERR_SHAPE, GRAFT_ERR_DTYPE, GRAFT_ERR_WORKSPACE, GRAFT_ERR_HIP = range(6)
GRAFT_STATUS_BAD_LENGTH, GRAFT_STATUS_BAD_TREE, GRAFT_STATUS_PATH_OVERFLOW = 1, 2, 4
GRAFT_F32, GRAFT_BF16 = 0, 1

_ERR_NAMES = {1: "GRAFT_ERR_NULL", 2: "GRAFT_ERR_SHAPE", 3: "GRAFT_ERR_DTYPE",
              4: "GRAFT_ERR_WORKSPACE", 5: "GRAFT_ERR_HIP"}

_i32, _i64, _f32, _vp, _sz = ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t
_SIGNATURES = {
    "graft_last_hip_error": (_i32, []),
    "graft_version": (_i32, []),
    "graft_retrieve": (_i32, [_vp, _vp, _i32, _i32, _vp, _vp, _i32, _i32, _i32, _i32, _i32,
                              _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "graft_build_tree_mask": (_i32, [_vp, _vp, _vp, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _i32, _vp, _vp]),
    "graft_tree_attn_workspace_bytes": (_sz, [_i32] * 7),
    "graft_tree_attn": (_i32, [_vp, _vp, _vp, _i64, _i64, _i64, _vp, _i32, _vp, _vp, _vp,
                               _i32, _i32, _i32, _i32, _i32, _i32, _f32, _i32, _vp, _vp, _sz, _vp]),
    "graft_attn_profile_events": (_i32, [_vp, _vp, _i32]),
    "graft_accept_workspace_bytes": (_sz, [_i32] * 3),
    "graft_accept": (_i32, [_vp, _vp, _vp, _vp, _i32, _vp, _i32, _i32, _i32,
                            _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "graft_accept_noalloc": (_i32, [_vp, _vp, _vp, _vp, _i32, _vp, _i32, _i32, _i32,
                                    _vp, _vp, _vp, _vp, _vp, _vp]),
    "graft_prune_select": (_i32, [_vp, _vp, _vp, _vp, _i32, _i32, _vp, _vp, _vp, _vp, _i32] + [_vp] * 8),
    "graft_matrix_retrieve": (_i32, [_vp, _i32, _i32, _vp, _vp, _i32, _vp, _i32, _i32, _vp, _vp, _vp, _vp, _vp]),
    "graft_matrix_update_workspace_bytes": (_sz, [_i32] * 4),
    "graft_matrix_update": (_i32, [_vp, _vp, _vp, _i32, _i32, _i32, _vp, _i32, _vp, _vp, _sz, _vp]),
    "graft_kv_compact": (_i32, [_vp, _vp, _i64, _i32, _i64, _i64, _i64, _vp, _i32, _vp, _vp, _vp,
                                _i32, _i32, _i32, _i32, _i32, _i32, _vp, _vp, _vp]),
}
EXPORTED_SYMBOLS = tuple(_SIGNATURES)

_lib = None
_bound = None          # the native marshalling module, once it has resolved the library


class GraftError(RuntimeError):
    def __init__(self, fn: str, code: int, hip: int = 0):
        self.code = code
        msg = "%s returned %s" % (fn, _ERR_NAMES.get(code, str(code)))
        if code == GRAFT_ERR_HIP:
            msg += " (hipError_t %d)" % hip
        super().__init__(msg)


def _built(path):
    if not os.path.exists(path):
        raise FileNotFoundError(
            "%s is missing: build it with `python -m paper_2605_20104_amd.build` "
            "(there is no fallback path)" % path)
    return path


def load_library():
    """dlopen libgraft.so and declare its signatures (the C ABI; the calls below also need _native.so).
    Raises if it has not been built."""
    global _lib
    if _lib is None:
        lib = ctypes.CDLL(_built(LIB_PATH))
        for name, (res, args) in _SIGNATURES.items():
            f = getattr(lib, name)
            f.restype, f.argtypes = res, args
        _lib = lib
    return _lib


def _calls():
    """The native marshalling functions, bound to the library."""
    global _bound
    if _bound is None:
        load_library()
        _built(NATIVE_PATH)
        from . import _native
        _native.bind(LIB_PATH, GraftError)
        _bound = _native
    return _bound


def graft_retrieve(ctx, ctx_len, n_min: int, n_max: int, C: int, m: int, tail=None, tail_len=None,
                   out=None, stream=None):
    """Ranked continuation chains of the suffix n-gram.  ctx int32 [B,L_max] on the GPU.

    Returns a dict of device tensors: chain_tok [B,C,m], chain_len, chain_pos,
    chain_match [B,C], n_hits [B], status [B].  `out` may carry preallocated ones.
    """
    return _calls().retrieve(ctx, ctx_len, n_min, n_max, C, m, tail, tail_len, out, stream)


def graft_build_tree_mask(parent, n_nodes, prefix_len, n_leaf_max: int = 0, depth_cap: int = 0,
                          out=None, stream=None):
    """Ancestor masks [B,K,2] (int64 storage of the uint64 words), pos, depth, optional leaf paths."""
    return _calls().build_tree_mask(parent, n_nodes, prefix_len, n_leaf_max, depth_cap, out, stream)


def graft_tree_attn_workspace_bytes(B: int, K_max: int, Hq: int, Hkv: int, D: int, max_pages: int,
                                    dtype: int) -> int:
    return int(load_library().graft_tree_attn_workspace_bytes(B, K_max, Hq, Hkv, D, max_pages, dtype))


def graft_tree_attn(q, k_cache, v_cache, strides, block_table, prefix_len, n_nodes, mask, Hkv: int,
                    scale: float, out=None, workspace=None, stream=None):
    """Tree-masked GQA attention, one layer.  q [B,K,Hq,D] float32 or bfloat16 on the GPU.

    strides: dict with 'page', 'token', 'head' in elements.  workspace: uint8 device
    tensor of at least graft_tree_attn_workspace_bytes(...) bytes (allocated if None).
    """
    return _calls().tree_attn(q, k_cache, v_cache, strides, block_table, prefix_len, n_nodes, mask, Hkv, scale,
                             out, workspace, stream)


def graft_accept_workspace_bytes(B: int, K_max: int, V: int) -> int:
    return int(load_library().graft_accept_workspace_bytes(B, K_max, V))


def graft_accept(parent, tokens, n_nodes, depth_cap: int, target_ids=None, logits=None, out=None,
                 workspace=None, stream=None):
    """Greedy acceptance walk.  Give target_ids int32 [B,K] or logits float32 [B,K,V] (then
    the argmax per node is returned in out['target_ids'])."""
    return _calls().accept(parent, tokens, n_nodes, depth_cap, target_ids, logits, out, workspace, stream)


def graft_accept_noalloc(parent, tokens, n_nodes, depth_cap: int, out, target_ids, logits=None, stream=None):
    """graft_accept without a workspace and without any allocation, here or in the library: every
    output tensor is the caller's (out: accept_len, best_node, path, out_tokens, status; target_ids
    is an input in target_ids mode and an output in logits mode)."""
    return _calls().accept_noalloc(parent, tokens, n_nodes, depth_cap, out, target_ids, logits, stream)


def graft_matrix_retrieve(M, tpl_parent, tpl_rank, n_ret, tokens, parent, n_nodes, status=None, stream=None):
    """Fills the first n_ret[b] template nodes by lookups in M [V,k] and appends them to the tree
    (tokens, parent [B,K_max] and n_nodes [B] are updated in place).  Returns status [B]."""
    return _calls().matrix_retrieve(M, tpl_parent, tpl_rank, n_ret, tokens, parent, n_nodes, status, stream)


def graft_matrix_update_workspace_bytes(B: int, K_max: int, V: int, k: int) -> int:
    return int(load_library().graft_matrix_update_workspace_bytes(B, K_max, V, k))


def graft_matrix_update(tokens, n_nodes, logits, M, target_ids=None, workspace=None, stream=None):
    """M[tokens[b,i]] <- ids of the k largest logits of node i (M [V,k] updated in place).
    Returns target_ids [B,K_max] (the greedy token per node)."""
    return _calls().matrix_update(tokens, n_nodes, logits, M, target_ids, workspace, stream)


def graft_kv_compact(k_cache, v_cache, layer_stride: int, n_layers: int, strides, block_table, prefix_len,
                     path, accept_len, K_max: int, Hkv: int, D: int, out=None, stream=None):
    """Moves the accepted path's keys/values behind the prefix in place (all n_layers layers).
    Returns dict(new_prefix_len [B], status [B])."""
    return _calls().kv_compact(k_cache, v_cache, layer_stride, n_layers, strides, block_table, prefix_len, path,
                              accept_len, K_max, Hkv, D, out, stream)


def graft_prune_select(parent, tokens, logq, n_nodes, chk_depth, chk_log_tau, chk_keep, chk_ret, out=None,
                       stream=None):
    """Confidence gates + selection of the retained draft nodes.  Returns a dict of device tensors:
    parent, tokens, index [B,K_max], n_nodes, stage, n_ret, status [B]."""
    return _calls().prune_select(parent, tokens, logq, n_nodes, chk_depth, chk_log_tau, chk_keep, chk_ret, out,
                                stream)
