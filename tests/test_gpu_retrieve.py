"""GPU parity: graft_retrieve vs the CPU oracle, bit-exact (runs on the MI355X only)."""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2605_20104_amd as graft
from gpu_util import assert_same, dev, host_dict, us_per_call

pytestmark = pytest.mark.gpu
KEYS = ("chain_tok", "chain_len", "chain_pos", "chain_match", "n_hits", "status")


def both(ctx, ctx_len, n_min, n_max, C, m, tail=None, tail_len=None):
    ref = oracle.retrieve(ctx, ctx_len, n_min, n_max, C, m, tail, tail_len)
    out = graft.graft_retrieve(dev(ctx), dev(ctx_len), n_min, n_max, C, m, dev(tail), dev(tail_len))
    return host_dict(out), ref


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c4", "c5"])
def test_workloads(name):
    w = inputs.get_workload(name)
    s = inputs.make_step_inputs(w)
    gpu, ref = both(s["ctx"], s["ctx_len"], w.n_min, w.n_max, w.C, w.m, s["tail"], s["tail_len"])
    assert_same(gpu, ref, KEYS)
    for b in range(w.B):                      # and they are the planted continuations
        assert gpu["chain_pos"][b].tolist() == s["planted_pos"][b][:w.C]


@pytest.mark.parametrize("seed", range(6))
def test_tiny_alphabet_many_overlaps(seed):
    rng = np.random.default_rng(seed)
    B, L_max = 5, int(rng.integers(40, 3000))
    vocab = int(rng.integers(2, 5))
    ctx = rng.integers(0, vocab, size=(B, L_max)).astype(np.int32)
    ctx_len = rng.integers(0, L_max + 1, size=B).astype(np.int32)
    ctx_len[0], ctx_len[1], ctx_len[2] = L_max, 0, 1
    tail = rng.integers(0, vocab, size=(B, 6)).astype(np.int32)
    tail_len = rng.integers(0, 7, size=B).astype(np.int32)
    n_min, n_max = int(rng.integers(1, 4)), int(rng.integers(4, 33))
    C, m = int(rng.integers(1, 9)), int(rng.integers(1, 20))
    use_tail = seed % 2 == 0
    gpu, ref = both(ctx, ctx_len, n_min, n_max, C, m, tail if use_tail else None,
                    tail_len if use_tail else None)
    assert_same(gpu, ref, KEYS)


def test_periodic_long_buffer_and_limits():
    ctx = np.full((2, 70000), 7, np.int32)            # every position is a hit; > one scan sweep
    ctx[1, ::3] = 8
    gpu, ref = both(ctx, [70000, 69999], 1, graft.GRAFT_MAX_NGRAM, graft.GRAFT_MAX_CHAINS, 5)
    assert_same(gpu, ref, KEYS)
    assert gpu["n_hits"][0] == 69999


def test_long_tail_and_query_in_every_place():
    """The query can lie in the tail alone, across the end of the context and the tail, or in the context
    beyond the first chunks; tails longer than a workgroup has threads are read from memory."""
    rng = np.random.default_rng(11)
    B, L_max, tail_max = 4, 40000, 1100
    ctx = rng.integers(0, 6, size=(B, L_max)).astype(np.int32)
    tail = rng.integers(0, 6, size=(B, tail_max)).astype(np.int32)
    ctx_len = np.array([40000, 33000, 16385, 5], np.int32)
    tail_len = np.array([1100, 3, 1060, 0], np.int32)
    gpu, ref = both(ctx, ctx_len, 2, 32, 8, 7, tail, tail_len)
    assert_same(gpu, ref, KEYS)
    assert gpu["status"].tolist() == [0, 0, 0, 0] and gpu["n_hits"][0] > 0


def test_no_hits_and_bad_lengths():
    ctx = np.arange(500, dtype=np.int32).reshape(1, 500).repeat(3, 0)
    gpu, ref = both(ctx, [500, 501, -1], 1, 4, 2, 4)
    assert_same(gpu, ref, KEYS)
    assert gpu["status"].tolist() == [0, graft.GRAFT_STATUS_BAD_LENGTH, graft.GRAFT_STATUS_BAD_LENGTH]
    assert (gpu["chain_tok"] == -1).all()


def test_outputs_fully_overwritten():
    """Stale output buffers must not leak through: run on dirty preallocated outputs."""
    w = inputs.get_workload("c2")
    s = inputs.make_step_inputs(w)
    ref = oracle.retrieve(s["ctx"], s["ctx_len"], w.n_min, w.n_max, 8, 12, s["tail"], s["tail_len"])
    out = {k: torch.full(tuple(ref[k].shape), 12345, dtype=torch.int32, device="cuda") for k in KEYS}
    graft.graft_retrieve(dev(s["ctx"]), dev(s["ctx_len"]), w.n_min, w.n_max, 8, 12, dev(s["tail"]),
                         dev(s["tail_len"]), out=out)
    assert_same(host_dict(out), ref, KEYS)


@pytest.mark.parametrize("n_min", [1, 2])
@pytest.mark.parametrize("L", [32768, 32769, 32770, 32771, 40960, 40961, 65537, 73731, 131075])
def test_contexts_around_and_beyond_the_ring(L, n_min):
    """Up to 32768 tokens the context is scanned in LDS, beyond that from registers, in units of 8192 tokens: matches that
    end at the edges of lanes, wavefronts, groups, units and of the row, rows that start at any element."""
    rng = np.random.default_rng(L + n_min)
    B, n_max = 3, 9
    query = rng.integers(100, 200, n_max).astype(np.int32)
    ctx = rng.integers(0, 100, size=(B, L)).astype(np.int32)
    ctx[2] = rng.integers(0, 4, L)                                     # and a row that is nothing but candidates
    ctx_len = np.array([L, L - 1, L - 2], np.int32)
    tail = np.zeros((B, n_max), np.int32)
    tail[:2], tail_len = query, np.array([n_max, n_max, 0], np.int32)
    ends = [0, 1, n_max - 1, 255, 256, 4095, 4096, 8191, 8192, 16383, 16384, 32767, 32768, L - 5, L - 4, L - 3, L - 2, L - 1]
    for b in range(2):
        for i in [i for i in (ends[b::2] if n_min == 1 else ends[1 - b::2]) if i < L]:
            k = int(min(i + 1, rng.integers(1, n_max + 1)))
            ctx[b, i - k + 1:i + 1] = query[n_max - k:]
    gpu, ref = both(ctx, ctx_len, n_min, n_max, 8, 6, tail, tail_len)
    assert_same(gpu, ref, KEYS)
    assert gpu["n_hits"][0] > 0 and gpu["n_hits"][2] > 1000


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 7, 257, 1023, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16387])
def test_rows_around_the_workgroup_sizes(L):
    """256 threads scan rows of up to 2048 tokens, 512 up to 8192, 1024 what is longer; the last group of four may be cut
    short, and the query may lie in context and tail."""
    rng = np.random.default_rng(L)
    B, n_max = 4, 6
    query = rng.integers(100, 200, n_max).astype(np.int32)
    ctx = rng.integers(0, 100, size=(B, L)).astype(np.int32)
    ctx[3] = rng.integers(0, 20, L)
    for b in range(3):
        for i in {0, 1, L // 3, L - 6, L - 3, L - 2, L - 1, 1023, 1024, 4094, 4095} & set(range(L)):
            k = int(min(i + 1, rng.integers(1, n_max + 1)))
            ctx[b, i - k + 1:i + 1] = query[n_max - k:]
    ctx_len = np.array([L, L - 1, max(0, L - 2), L], np.int32)
    tail = np.tile(query, (B, 60)).astype(np.int32)                    # 360 tokens: more than the smallest workgroup has threads
    tail_len = np.array([360, 6, 3, 0], np.int32)
    for n_min in (1, 2):
        gpu, ref = both(ctx, ctx_len, n_min, n_max, 8, 6, tail, tail_len)
        assert_same(gpu, ref, KEYS)


@pytest.mark.parametrize("hits", [0, 1, 7, 8, 9, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("L", [4096, 8192, 20000])
def test_as_many_hits_as_the_ranking_list_holds(L, hits):
    rng = np.random.default_rng(hits)
    ctx = rng.integers(0, 100, size=(1, L)).astype(np.int32)
    for at in rng.permutation(L // 16 - 1)[:hits]:                     # one hit a thread at most, of one to five tokens
        ctx[0, 16 * at + 9] = 300
        for k in range(int(rng.integers(0, 5))):
            ctx[0, 16 * at + 8 - k] = 299 - k
    tail = np.array([[296, 297, 298, 299, 300]], np.int32)
    for C, m in ((3, 8), (8, 20)):                                     # (160 tokens: three wavefronts write)
        gpu, ref = both(ctx, np.array([L], np.int32), 1, 5, C, m, tail, np.array([5], np.int32))
        assert_same(gpu, ref, KEYS)
        assert gpu["n_hits"][0] == hits


@pytest.mark.parametrize("n_max", [2, 8, 9, 10, 17, 31, 32])
def test_long_matches_across_the_pieces_of_a_streamed_context(n_max):
    """A context that does not fit LDS is compared in pieces of 256 tokens of one wavefront and the 32 in front: matches of
    every length that end at the first tokens of a piece, a unit and the context, alone and one next to the other."""
    rng = np.random.default_rng(n_max)
    L, tail = 60000, np.tile(rng.integers(100, 110, n_max).astype(np.int32), (4, 1))
    ctx = rng.integers(0, 100, size=(4, L)).astype(np.int32)
    for b, starts in enumerate(([0, 256, 4096, 32768], [512, 3840, 8192, 40960], [8448, 36864, 45056, L - 40])):
        for start in starts:
            for i in range(start + b, start + 39, 3):              # (a later match overwrites part of an earlier one)
                k = int(min(i + 1, rng.integers(1, n_max + 1)))
                ctx[b, i - k + 1:i + 1] = tail[b, n_max - k:]
    ctx[3], tail[3] = 5, 5                                          # and one token all along
    gpu, ref = both(ctx, np.full(4, L, np.int32), 1, n_max, 8, 6, tail, np.full(4, n_max, np.int32))
    assert_same(gpu, ref, KEYS)
    assert (gpu["n_hits"] > 10).all()


def test_repetitive_contexts_take_as_long_beyond_the_ring():
    """One token all along, nothing but candidates: per token, a context that does not fit LDS takes about as long as one that
    does (2.5 times as long with a trip to memory for every candidate)."""
    def us(L):
        ctx, length = dev(np.full((1, L), 7)), dev([L])
        out = graft.graft_retrieve(ctx, length, 2, 32, 3, 8)
        return us_per_call(lambda stream: graft.graft_retrieve(ctx, length, 2, 32, 3, 8, out=out, stream=stream)) / L
    inside, beyond = us(32768), us(65536)
    assert beyond < 1.5 * inside, (inside, beyond)


def test_repetitive_rows_of_4096_tokens_take_a_larger_workgroup():
    """One token all along: a thread compares its tokens one after the other, and 16 of them in each thread of a workgroup of
    256 take 1.33 times as long as slightly longer rows in one of 512."""
    def us(L):
        ctx, length = dev(np.full((1, L), 7)), dev([L])
        out = graft.graft_retrieve(ctx, length, 2, 32, 3, 8)
        return us_per_call(lambda stream: graft.graft_retrieve(ctx, length, 2, 32, 3, 8, out=out, stream=stream))
    below, above = us(4096), us(4100)
    assert below < 1.2 * above, (below, above)
