"""The native marshalling of the Python binding (no GPU): arguments that do not fit are Python errors,
argument errors of the library are GraftError, and nothing is launched in either case."""
import sys

import pytest
import torch

import paper_2605_20104_amd as graft


def _mask(parent=None, n_leaf_max=4, depth_cap=200, out=None):
    one = torch.ones(2, dtype=torch.int32)
    parent = torch.zeros((2, 8), dtype=torch.int32) if parent is None else parent
    return graft.graft_build_tree_mask(parent, one, one, n_leaf_max, depth_cap, out=out, stream=0)


@pytest.mark.parametrize("kwargs,error", [
    (dict(parent=torch.zeros((8, 2), dtype=torch.int32).t()), AssertionError),       # not dense row-major
    (dict(parent=torch.zeros(8, dtype=torch.int32)), ValueError),                    # not [B, K]
    (dict(parent=3), TypeError),
    (dict(out={}), KeyError),                                                        # an output is missing
    (dict(n_leaf_max="4"), TypeError),
])
def test_arguments_that_do_not_fit(kwargs, error):
    with pytest.raises(error):
        _mask(**kwargs)


def test_logits_are_three_dimensional():
    one = torch.ones(1, dtype=torch.int32)
    for shape in ((1, 4, 8, 1), (4, 8)):
        with pytest.raises(ValueError):
            graft.graft_matrix_update(torch.zeros((1, 4), dtype=torch.int32), one, torch.zeros(shape), torch.zeros((8, 2), dtype=torch.int32),
                                      stream=0)


def test_library_errors_carry_their_code():
    with pytest.raises(graft.GraftError) as e:
        _mask(depth_cap=200)
    assert e.value.code == graft.GRAFT_ERR_SHAPE and "graft_build_tree_mask" in str(e.value)
    q = torch.zeros((1, 4, 8, 96), dtype=torch.bfloat16)
    with pytest.raises(graft.GraftError) as e:
        graft.graft_tree_attn(q, q, q, {"page": 1536, "token": 96, "head": 96}, torch.zeros((1, 2), dtype=torch.int32), *(
            [torch.zeros(1, dtype=torch.int32)] * 2), torch.zeros((1, 4, 2), dtype=torch.int64), 2, 0.1, stream=0)
    assert e.value.code == graft.GRAFT_ERR_SHAPE
    with pytest.raises(AssertionError):                                               # mixed storage types
        graft.graft_tree_attn(q, q.float(), q, {"page": 1, "token": 1, "head": 1}, torch.zeros((1, 2), dtype=torch.int32),
                              None, None, None, 2, 0.1, stream=0)


def test_strides_from_a_mapping_that_makes_its_values():
    """The values are held while they are read: they die behind it, not before."""
    events = []

    class Value:
        def __int__(self):
            events.append("read")
            return 12

        def __del__(self):
            events.append("gone")

    class Strides:
        def __getitem__(self, key):
            return Value()

    q = torch.zeros((1, 4, 8, 64), dtype=torch.bfloat16)
    one = torch.zeros(1, dtype=torch.int32)
    with pytest.raises(graft.GraftError) as e:                                        # 12 is no stride of D = 64
        graft.graft_tree_attn(q, q, q, Strides(), torch.zeros((1, 2), dtype=torch.int32), one, one,
                              torch.zeros((1, 4, 2), dtype=torch.int64), 2, 0.1, stream=0)
    assert e.value.code == graft.GRAFT_ERR_SHAPE and events == ["read"] * 3 + ["gone"] * 3


def test_the_c_abi_loads_without_the_native_module(monkeypatch):
    """Users of the C ABI alone need libgraft.so alone; the Python calls say what to build."""
    monkeypatch.setattr(graft, "_lib", None)
    monkeypatch.setattr(graft, "_bound", None)
    monkeypatch.setattr(graft, "NATIVE_PATH", "/nonexistent/_native.so", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2605_20104_amd._native", None)             # as if it were not there
    monkeypatch.delattr(graft, "_native", raising=False)
    assert graft.load_library().graft_version() >= 100
    assert graft.graft_accept_workspace_bytes(1, 16, 1000) > 0
    with pytest.raises(FileNotFoundError, match="paper_2605_20104_amd.build"):
        _mask()


@pytest.mark.gpu
def test_out_of_memory_is_torchs_own_error():
    ctx, n = torch.zeros((1, 8), dtype=torch.int32, device="cuda"), torch.full((1,), 8, dtype=torch.int32, device="cuda")
    with pytest.raises(torch.OutOfMemoryError):                                       # 4 TiB of results, refused by the allocator
        graft.graft_retrieve(ctx, n, 1, 4, 1 << 20, 1 << 20)


def _attention(seed, B=1, K=20, H=4, D=64, pages=300):
    """fp32, head size 64, a prefix long enough that the keys are split: (arguments, bytes of workspace)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.randn((B, K, H, D), generator=gen, device="cuda")
    k, v = (torch.randn((pages, H, 16, D), generator=gen, device="cuda") for _ in range(2))
    table = torch.randperm(pages, generator=gen, device="cuda").to(torch.int32)[None].contiguous()
    n, prefix = torch.full((B,), K, dtype=torch.int32, device="cuda"), torch.full((B,), pages * 16 - K, dtype=torch.int32, device="cuda")
    parent = torch.arange(-1, K - 1, dtype=torch.int32, device="cuda")[None].contiguous()
    mask = graft.graft_build_tree_mask(parent, n, prefix)["mask"]
    need = graft.graft_tree_attn_workspace_bytes(B, K, H, H, D, pages, graft.GRAFT_F32)
    return (q, k, v, {"page": H * 16 * D, "token": D, "head": 16 * D}, table, prefix, n, mask, H, 0.125), need


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["attention", "accept", "matrix_update"])
def test_workspace_belongs_to_the_stream_of_the_call(call):
    """The block of a workspace that the call allocates is in a segment of the stream the kernels run on."""
    one = torch.full((1,), 16, dtype=torch.int32, device="cuda")
    tree = torch.arange(-1, 15, dtype=torch.int32, device="cuda")[None].contiguous()
    logits = torch.randn((1, 16, 5000), device="cuda")
    M = torch.full((5000, 8), -1, dtype=torch.int32, device="cuda")
    args, need = _attention(1)
    if call != "attention":
        need = graft.graft_accept_workspace_bytes(1, 16, 5000) if call == "accept" else graft.graft_matrix_update_workspace_bytes(1, 16, 5000, 8)
    assert need > 0
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    on_side = lambda: sum(s["total_size"] for s in torch.cuda.memory_snapshot() if s["stream"] == side.cuda_stream)
    before = on_side()
    if call == "attention":
        graft.graft_tree_attn(*args, stream=side)
    elif call == "accept":
        graft.graft_accept(tree, tree, one, 8, logits=logits, stream=side)
    else:
        graft.graft_matrix_update(tree, one, logits, M, stream=side.cuda_stream)     # the handle itself
    torch.cuda.synchronize()
    assert side.cuda_stream != torch.cuda.current_stream().cuda_stream and on_side() - before >= need


@pytest.mark.gpu
def test_calls_on_two_streams_without_a_workspace():
    """Calls in flight on two streams keep their partial results apart: the bits are those of calls one by one."""
    problems = [_attention(s)[0] for s in (2, 3)]
    alone = [graft.graft_tree_attn(*p) for p in problems]
    streams = [torch.cuda.Stream() for _ in problems]
    outs = [[torch.empty_like(a) for _ in range(20)] for a in alone]
    torch.cuda.synchronize()
    for i in range(20):
        for p, s, o in zip(problems, streams, outs):
            graft.graft_tree_attn(*p, out=o[i], stream=s)
    torch.cuda.synchronize()
    for a, o in zip(alone, outs):
        for x in o:
            assert torch.equal(a, x)
    assert torch.equal(graft.graft_tree_attn(*problems[0], stream=0), alone[0])          # the null stream, by its handle
