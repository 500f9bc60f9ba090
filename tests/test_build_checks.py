"""The build checks the generated assembly of the hand-scheduled attention kernels.  These tests
feed the checker small assembly texts with one planted mistake each (on the CPU), and run it
over the assembly of the library that is actually built."""
import os
import re

import pytest

from paper_2605_20104_amd import build as b

KERNEL = "_ZN5graft21tree_attn_mfma_kernelILi2EEEvNS_10AttnParamsE"


def _asm(body, scratch=0):
    return "\n".join([
        "\t.text",
        KERNEL + ":",
        "\ts_load_dwordx2 s[0:1], s[4:5], 0x0",
        body,
        "\ts_endpgm",
        "\t.amdhsa_kernel " + KERNEL,
        "\t\t.amdhsa_private_segment_fixed_size %d" % scratch,
        "\t.end_amdhsa_kernel",
        ".Lfunc_end0:",
    ])


MFMA = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[10:13], v[20:23], a[0:3]\n\t;;#ASMEND"
MFMA_C = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 v[40:43], v[10:13], a[96:99], v[30:33]\n\t;;#ASMEND"
FILL = "\tv_add_u32_e32 v1, v2, v3\n\ts_add_i32 s0, s1, s2"


def test_clean_text_passes():
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA + "\n" + MFMA_C)) == []


@pytest.mark.parametrize("writer", ["v_mov_b32_e32 v11, v5", "v_cvt_pk_bf16_f32 v23, v1, v2",
                                    "v_mov_b64_e32 v[12:13], s[2:3]", "v_accvgpr_read_b32 v20, a200"])
def test_vector_write_of_a_source_right_before_the_mfma(writer):
    bad = b.check_attention_asm(_asm(FILL + "\n\t" + writer + "\n" + MFMA))
    assert len(bad) == 1 and "MFMA source" in bad[0]
    # one instruction in between is one wait state: still too close
    assert b.check_attention_asm(_asm(FILL + "\n\t" + writer + "\n\ts_add_i32 s0, s1, s2\n" + MFMA))
    # two wait states are enough, as two instructions or as s_nop 1
    assert b.check_attention_asm(_asm("\t" + writer + "\n" + FILL + "\n" + MFMA)) == []
    assert b.check_attention_asm(_asm("\t" + writer + "\n\ts_nop 1\n" + MFMA)) == []
    assert b.check_attention_asm(_asm("\t" + writer + "\n\ts_nop 0\n" + MFMA))


def test_accumulator_input_in_vgprs_is_a_source_too():
    assert b.check_attention_asm(_asm(FILL + "\n\tv_mov_b32_e32 v31, 0\n" + MFMA_C))
    assert b.check_attention_asm(_asm(FILL + "\n\tv_mov_b32_e32 v50, 0\n" + MFMA_C)) == []


def test_writes_that_are_not_vector_registers_do_not_count():
    ok = FILL + "\n\tv_cmp_gt_f32_e32 vcc, v10, v11\n\tv_readfirstlane_b32 s3, v20\n" + MFMA
    assert b.check_attention_asm(_asm(ok)) == []


def test_unknown_predecessor_after_a_label():
    assert b.check_attention_asm(_asm(FILL + "\n.LBB0_3:\n" + MFMA))
    assert b.check_attention_asm(_asm(FILL + "\n.LBB0_3:\n\ts_nop 1\n" + MFMA)) == []


def test_compiler_use_of_a_hand_managed_accvgpr():
    # 48 * MB + 4 * min(MB, 4) = 104 registers are hand-managed in the MB = 2 kernel
    bad = b.check_attention_asm(_asm(FILL + "\n\tv_accvgpr_write_b32 a103, v1\n" + FILL))
    assert len(bad) == 1 and "AccVGPR" in bad[0]
    assert b.check_attention_asm(_asm(FILL + "\n\tds_read_b32 a17, v1\n" + FILL))
    assert b.check_attention_asm(_asm(FILL + "\n\tv_accvgpr_write_b32 a104, v1\n" + FILL)) == []
    inside = "\t;;#ASMSTART\n\tv_accvgpr_write_b32 a[5], v1\n\t;;#ASMEND"
    assert b.check_attention_asm(_asm(FILL + "\n" + inside)) == []


NOPS = "\ts_nop 7\n\ts_nop 3"          # 8 + 4 = 12 wait states


@pytest.mark.parametrize("reader", ["v_exp_f32_e32 v1, v41", "v_max3_f32 v2, v3, v40, v43", "ds_write_b32 v5, v42",
                                    "global_store_dwordx4 v[6:7], v[40:43], off", "v_cmp_gt_f32_e32 vcc, v40, v1",
                                    "v_accvgpr_write_b32 a200, v43"])
def test_read_of_an_mfma_result_in_vgprs_too_early(reader):
    bad = b.check_attention_asm(_asm(FILL + "\n" + MFMA_C + "\n\t" + reader))
    assert len(bad) == 1 and "MFMA result" in bad[0]
    # eleven wait states are not enough, twelve are; a label in between does not reset the count
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA_C + "\n\ts_nop 7\n\ts_nop 2\n\t" + reader))
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA_C + "\n" + NOPS + "\n\t" + reader)) == []
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA_C + "\n\ts_nop 3\n.LBB0_7:\n\t" + reader))
    # registers next to the result are not the result
    other = reader.replace("v40", "v39").replace("v41", "v44").replace("v42", "v44").replace("v43", "v44") \
                  .replace("v[40:43]", "v[44:47]")
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA_C + "\n\t" + other)) == []


def test_read_of_an_accumulator_too_early():
    rd = "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v1, a[2]\n\t;;#ASMEND"
    bad = b.check_attention_asm(_asm(FILL + "\n" + MFMA + "\n" + rd))
    assert len(bad) == 1 and "MFMA result" in bad[0]
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA + "\n" + NOPS + "\n" + rd)) == []
    # another MFMA accumulating into the same registers is not such a reader
    assert b.check_attention_asm(_asm(FILL + "\n" + MFMA + "\n" + MFMA)) == []


def test_accvgpr_write_of_a_source_right_before_the_mfma():
    wr = "\t;;#ASMSTART\n\tv_accvgpr_write_b32 a[97], v1\n\t;;#ASMEND"
    bad = b.check_attention_asm(_asm(FILL + "\n" + wr + "\n" + MFMA_C))
    assert len(bad) == 1 and "MFMA source" in bad[0]
    assert b.check_attention_asm(_asm(FILL + "\n" + wr + "\n\ts_nop 1\n" + MFMA_C)) == []


def test_scratch_memory():
    bad = b.check_attention_asm(_asm(FILL, scratch=128))
    assert len(bad) == 1 and "scratch" in bad[0]


# no stages: straight to the exchange; else the loop, which ends with a wait
TRANSFERS = """\t;;#ASMSTART
\tbuffer_load_dwordx4 v3, s[0:3], 0 offen lds
\t;;#ASMEND
\ts_cbranch_scc1 .LBB0_2
%s
.LBB0_1:
\ts_nop 1
""" + MFMA + """
\ts_cbranch_scc1 .LBB0_1
\ts_waitcnt vmcnt(0)
.LBB0_2:
%s
\ts_barrier
\tds_write_b128 v1, v[2:5]
\ts_endpgm"""


@pytest.mark.parametrize("transfer", ["buffer_load_dwordx4 v3, s[0:3], 0 offen lds", "global_load_lds_dword v[4:5], off"])
def test_lds_written_while_a_transfer_may_be_in_flight(transfer):
    def check(in_front, at_exchange):
        return b.check_attention_asm(_asm(TRANSFERS.replace("buffer_load_dwordx4 v3, s[0:3], 0 offen lds", transfer) % (in_front, at_exchange)))

    bad = check("\ts_nop 0", "\ts_nop 0")                        # nothing waits on the path around the loop
    assert len(bad) == 1 and "in flight" in bad[0] and "ds_write_b128" in bad[0]
    assert len(check("\ts_waitcnt vmcnt(8)", "\ts_nop 0")) == 1
    assert len(check("\ts_nop 0", "\ts_waitcnt vmcnt(1) lgkmcnt(0)")) == 1
    assert check("\ts_nop 0", "\ts_waitcnt vmcnt(0) lgkmcnt(0)") == []
    # the wavefront's own wait says nothing about the others' without a barrier behind it
    assert len(check("\ts_nop 0", "\ts_barrier\n\ts_waitcnt vmcnt(0)\n\tds_write_b32 v1, v2")) == 1
    # LDS writes from which the loop is still to come are its own affair
    assert check("\tds_write_b128 v1, v[2:5]", "\ts_waitcnt vmcnt(0)") == []


@pytest.mark.parametrize("source,mfma", [("tree_attn.hip", "v_mfma_f32_16x16x32_bf16"), ("tree_attn_wide.hip", "v_mfma_f32_32x32x16_bf16")])
def test_the_built_library_passes(source, mfma):
    path = b._asm_of(source)
    if not os.path.exists(path):
        pytest.skip("no assembly kept from a build in this tree")
    with open(path) as f:
        text = f.read()
    assert text.count(mfma) > 500                                # the check sees the real kernels
    assert b.check_attention_asm(text) == []


@pytest.mark.parametrize("splits", [2, 4, 8, 16])
def test_the_merge_picks_its_scales_by_value(splits):
    """Partial rows in 32-row blocks have two scales, one for either half of the dims.  Picked as one of two elements of the
    splits' array they became a chain of selects over all of it, for every split: 275 instructions for 23, 2.4 us of 7.6."""
    path = b._asm_of("tree_attn.hip")
    if not os.path.exists(path):
        pytest.skip("no assembly kept from a build in this tree")
    with open(path) as f:
        text = f.read()
    selects = [len(re.findall(r"v_cndmask", re.search(r"^_ZN5graft24tree_attn_combine_kernelILi%dELb%dE\w*:(.*?)^\.Lfunc_end" % (splits, wide), text, re.M | re.S).group(1)))
               for wide in (0, 1)]
    assert selects[1] <= selects[0] + 2 * splits, selects


def test_no_kernel_of_the_library_uses_scratch_memory():
    """The kernels' metadata in the built library: an array or a register that went to scratch memory is a trip to memory
    for every access.  (The value behind the key is a small number, one byte, or marked as a larger one.)"""
    if not os.path.exists(b.LIB):
        b.build()
    with open(b.LIB, "rb") as f:
        data = f.read()
    key = b".private_segment_fixed_size"
    sizes = [data[at.end()] for at in re.finditer(re.escape(key), data)]
    assert len(sizes) >= len(b.SOURCES)
    assert set(sizes) == {0}, sizes


# ---- waits that count the requests behind a transfer
COUNTED = "_ZN5graft22tree_attn_parts_kernelILi64EEEvPKiS2_"
MORE = "\ts_cmp_ge_i32 s4, s5\n\ts_cselect_b64 s[6:7], -1, 0\n\ts_and_b64 vcc, exec, s[6:7]\n\ts_cbranch_vccnz .LBB0_%d"
LOOP = """\tglobal_load_lds_dwordx4 v1, s[0:1]
\tglobal_load_dwordx4 v[2:5], v1, s[2:3]
\tglobal_load_dwordx4 v[6:9], v1, s[2:3]
.LBB0_1:
\t;;#ASMSTART
\ts_waitcnt vmcnt(2)
\t;;#ASMEND
\tds_read_b128 v[20:23], v0
\tv_mfma_f32_32x32x16_f16 v[40:55], v[20:23], v[24:27], v[40:55]
\ts_waitcnt vmcnt(0)
%(first)s
\tglobal_load_lds_dwordx4 v1, s[0:1]
.LBB0_2:
\tv_mfma_f32_32x32x16_f16 v[40:55], v[2:5], v[6:9], v[40:55]
%(second)s
\tglobal_load_dwordx4 v[2:5], v1, s[2:3]
%(last)s
.LBB0_3:
%(back)s
\ts_branch .LBB0_1
.LBB0_4:
%(end)s
\tds_write_b128 v0, v[40:43]"""
WAY = dict(first=MORE % 2, second="\ts_and_b64 vcc, exec, s[6:7]\n\ts_cbranch_vccnz .LBB0_3", last="\tglobal_load_dwordx4 v[6:9], v1, s[2:3]",
           back="\ts_cmp_lt_i32 s4, s5\n\ts_cbranch_scc0 .LBB0_4", end="\ts_barrier")


def _counted(**other):
    return b.check_attention_asm(_asm(LOOP % dict(WAY, **other)).replace(KERNEL, COUNTED))


def test_a_wait_that_counts_the_requests_behind_a_transfer():
    assert _counted() == []
    assert _counted(last="\tbuffer_store_dword v6, v1, s[0:3], 0 offen") == []           # what is stored counts too
    # a load too few, in the loop or in front of it
    bad = _counted(last="\ts_nop 0")
    assert len(bad) == 1 and "only 1 requests" in bad[0]
    assert any("only 0 requests" in x for x in _counted(last="\tglobal_load_lds_dwordx4 v1, s[0:1]"))
    # a shorter wait in between is enough
    assert _counted(last="\ts_waitcnt vmcnt(1)") == []
    assert _counted(last="\ts_waitcnt lgkmcnt(0)") != []


def test_paths_that_a_condition_allows():
    # the loads behind the transfer go by another condition, or by one whose registers are others by then
    other = "\ts_and_b64 vcc, exec, s[8:9]\n\ts_cbranch_vccnz .LBB0_3"
    assert any("only 0 requests" in x for x in _counted(second=other))
    for write in ("\ts_mov_b64 s[6:7], s[8:9]", "\tv_cmp_gt_f32_e64 s[6:7], v1, v2", "\ts_add_i32 s7, s8, 1"):
        assert any("only 0 requests" in x for x in _counted(second=write + "\n" + WAY["second"]))
    assert _counted(second=WAY["second"].replace("s_and_b64", "s_andn2_b64")) != []
    # the same condition the other way round, and another compare of the same numbers
    inverse = "\ts_cmp_lt_i32 s4, s5\n\ts_cselect_b64 s[8:9], -1, 0\n\ts_andn2_b64 vcc, exec, s[8:9]\n\ts_cbranch_vccnz .LBB0_3"
    assert _counted(second=inverse) == []
    assert _counted(second="\ts_add_i32 s4, s4, 1\n" + inverse) != []                     # of other numbers
    assert _counted(second="\ts_cmp_gt_i32 s5, s4\n\ts_cbranch_scc0 .LBB0_3") == []


def test_the_exchange_behind_counted_transfers():
    bad = _counted(end="\ts_nop 0")
    assert len(bad) == 1 and "in flight" in bad[0]
    # the loop is left with a transfer that nobody has waited for
    assert any("in flight" in x for x in _counted(back="\ts_cbranch_execz .LBB0_4"))
    assert "no wait" in b.check_attention_asm(_asm((LOOP % WAY).replace(";;#ASMSTART", "").replace(";;#ASMEND", "")).replace(KERNEL, COUNTED))[0]


def test_the_waits_of_the_built_library():
    path = b._asm_of("tree_attn_parts.hip")
    if not os.path.exists(path):
        pytest.skip("no assembly kept from a build in this tree")
    with open(path) as f:
        text = f.read()
    assert text.count("global_load_lds_dwordx4") > 50 and b.check_attention_asm(text) == []
    # one of the sixteen loads behind a tile's transfers goes: the first of every run of sixteen, one at a time (the first tile's are
    # waited for in front of the loop, so that it can do without)
    lines, run, starts = text.split("\n"), 0, []
    for i, line in enumerate(lines):
        if line.startswith("\tglobal_load_lds"):
            run = 1
        elif run and line.startswith("\tglobal_load_dwordx"):
            starts.append(i)
            run = 0
    assert len(starts) == 8                                      # first tile, first of a table register's, loop and second pass, D = 64 and 128
    missed = [lines[i] for i in starts if not any("only 15 requests" in x for x in b.check_attention_asm("\n".join(lines[:i] + lines[i + 1:])))]
    assert len(missed) <= 2, missed
