"""Builds libgraft.so (the C-ABI library) from the HIP sources with hipcc for gfx950, and _native.so
(the native half of the Python binding, host code only) with g++."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJ_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libgraft.so")
LIB_TIMING = os.path.join(PKG, "libgraft_timing.so")     # the same library with the attention kernel's time stamps
NATIVE = os.path.join(PKG, "_native.so")                 # tensor marshalling of the Python binding (csrc/binding.cpp)
SOURCES = ["api.hip", "retrieve.hip", "tree_mask.hip", "tree_attn.hip", "tree_attn_wide.hip", "tree_attn_wide_128.hip", "tree_attn_direct.hip", "tree_attn_parts.hip", "accept.hip", "matrix.hip", "kv_compact.hip", "prune.hip"]

# packed-fp32 code generation is switched off for every device compile; VGPR spills must not
# land in AccVGPRs (the attention kernel manages those by hand).  Kernel arguments: the first 14 words arrive in
# scalar registers with the wavefront instead of being loaded by it, a cold trip to memory in front of every kernel's
# first request (0.4 us a launch: a round of four small kernels 19.0 -> 18.5 us, a layer's attention and merge with 2K keys
# 15.0 -> 14.0), so kernels take what that request needs first.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC,
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-mllvm", "-amdgpu-spill-vgpr-to-agpr=0", "-mllvm", "-amdgpu-kernarg-preload-count=16",
               "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


HAND_SCHEDULED = ["tree_attn.hip", "tree_attn_wide.hip", "tree_attn_wide_128.hip", "tree_attn_parts.hip"]     # their device assembly is kept and checked


def _asm_of(src: str, directory: str = OBJ_DIR) -> str:
    return os.path.join(directory, os.path.splitext(src)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")


def _compile(src: str, extra):
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    return _compile_to(src, extra, obj)


def _compile_to(src: str, extra, obj: str):
    keep = ["-save-temps=obj"] if src in HAND_SCHEDULED else []    # keeps the device assembly for the check below
    cmd = [_hipcc(), *HIPCC_FLAGS, *extra, *keep, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stdout))
    warn = [l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    return obj, "\n".join(warn)


def _reg_span(tok: str):
    """'v12' -> ('v', 12, 12); 'a[4:7]' -> ('a', 4, 7); 'a[0xf0]' -> ('a', 240, 240); else None."""
    m = re.fullmatch(r"([va])(\d+|0x[0-9a-f]+)", tok)
    if m:
        n = int(m.group(2), 0)
        return m.group(1), n, n
    m = re.fullmatch(r"([va])\[(\d+|0x[0-9a-f]+):(\d+|0x[0-9a-f]+)\]", tok)
    if m:
        return m.group(1), int(m.group(2), 0), int(m.group(3), 0)
    m = re.fullmatch(r"([va])\[(\d+|0x[0-9a-f]+)\]", tok)
    if m:
        n = int(m.group(2), 0)
        return m.group(1), n, n
    return None


def _managed_accvgprs(symbol: str) -> int:
    """AccVGPRs that a kernel manages by hand: tree_attn_mfma_kernel<MB>, tree_attn_wide_kernel<NB, MODE> or tree_attn_wide_128_kernel<NB, MODE>;
    None for others."""
    m = re.match(r"_ZN5graft21tree_attn_mfma_kernelILi(\d+)E", symbol)
    if m:
        mb = int(m.group(1))
        return 48 * mb + 4 * min(mb, 4)
    m = re.match(r"_ZN5graft\d+tree_attn_wide(?:_128)?_kernelILi(\d+)E", symbol)
    return 64 * int(m.group(1)) + 64 if m else None


# Wait states between an MFMA and the first other instruction that may read its result: the
# passes of the widest MFMA used here (8) plus 3, as for the compiler's own MFMAs, plus one.
MFMA_RESULT_WAIT = 12


def check_attention_asm(asm_text: str):
    """Checks the generated device assembly of the MFMA attention kernels against the rules
    their hand-placed registers and inline-assembly MFMAs rely on.  Returns a list of
    violations (empty = fine):
      * no scratch memory (register spills) in any of the kernels;
      * outside the inline-assembly blocks no instruction names a hand-managed AccVGPR
        (_managed_accvgprs: accumulators, Q operand, row sums);
      * no MFMA has a vector ALU instruction writing one of its VGPR sources within the two
        preceding wait states (an s_nop k counts k + 1): the hardware needs them and the
        compiler does not know that the asm statement is an MFMA.  The same holds for a
        v_accvgpr_write of an AccVGPR source;
      * no instruction other than an MFMA reads a register that an MFMA wrote within the
        MFMA_RESULT_WAIT preceding wait states, in program order across labels (the result of a
        MFMA is written at the end of its passes, and nothing interlocks a vector ALU,
        LDS or memory instruction, or a v_accvgpr_read, that comes earlier).  An MFMA issues no sooner
        than the one in front of it has gone through its passes: those count as wait states too;
      * the transfers from memory to LDS have landed where LDS gets another use (_check_transfers), and in tree_attn_parts_kernel
        where its keys are read (_check_counted_waits).
    """
    problems = _check_transfers(asm_text)
    lines = asm_text.split("\n")
    kernel, managed, in_asm, desc = None, 0, False, ""
    history = []          # (wait states, destination span or None) of the preceding instructions
    results = []          # [wait states since, span] of MFMA results still inside MFMA_RESULT_WAIT
    last_mfma = [0, 0]    # passes of the last MFMA, wait states since

    def age(states):
        last_mfma[1] += states
        for r in results:
            r[0] += states
        while results and results[0][0] >= MFMA_RESULT_WAIT:
            del results[0]

    for ln, raw in enumerate(lines, 1):
        text = raw.split(";")[0].strip() if not raw.lstrip().startswith(";") else ""
        m = re.match(r"^(_Z\w+):", raw)
        if m and _managed_accvgprs(m.group(1)):
            kernel, managed, history, results = m.group(1), _managed_accvgprs(m.group(1)), [(1, ("v", 0, 1 << 20))], []
            last_mfma[:] = [0, 0]
            continue
        if kernel and raw.startswith(".Lfunc_end"):
            kernel = None
            continue
        if "ASMSTART" in raw:
            in_asm = True
            continue
        if "ASMEND" in raw:
            in_asm = False
            continue
        m = re.match(r"\s*\.amdhsa_kernel\s+(\S+)", raw)
        if m:
            desc = m.group(1)
            continue
        m = re.match(r"\s*\.amdhsa_private_segment_fixed_size\s+(\d+)", raw)
        if m:
            if _managed_accvgprs(desc) and int(m.group(1)) != 0:
                problems.append("%s uses %s bytes of scratch memory (spills)" % (desc, m.group(1)))
            continue
        if not kernel:
            continue
        if raw.startswith(".LBB") or raw.startswith(".Ltmp"):
            if raw.startswith(".LBB"):
                # another block may jump here: assume that its last instruction wrote every VGPR
                history = [(1, ("v", 0, 1 << 20))]
            continue
        if not text or text.startswith("."):
            continue
        parts = text.replace(",", " ").split()
        op, args = parts[0], parts[1:]
        if not in_asm:
            for a in args:
                sp = _reg_span(a)
                if sp and sp[0] == "a" and sp[1] < managed:
                    problems.append("line %d (%s): compiler-generated use of a hand-managed AccVGPR: %s"
                                    % (ln, kernel, text))
        if op.startswith("v_mfma"):
            srcs = [sp for sp in map(_reg_span, args[1:]) if sp]
            states = 0
            for w, dst in reversed(history):
                if states >= 2:
                    break
                if dst is not None and any(dst[0] == s_[0] and dst[1] <= s_[2] and s_[1] <= dst[2] for s_ in srcs):
                    problems.append("line %d (%s): vector ALU write of an MFMA source %d wait state(s) before: %s"
                                    % (ln, kernel, states, text))
                    break
                states += w
            history.append((1, None))
            age(max(1, last_mfma[0] - last_mfma[1]))
            last_mfma[:] = [8 if "32x32" in op else 4, 0]
            d = _reg_span(args[0]) if args else None
            if d:
                results.append([0, d])
            continue
        if op == "s_nop":
            history.append((int(args[0], 0) + 1, None))
            age(int(args[0], 0) + 1)
            continue
        # any other instruction: it must not read what an MFMA has just written (stores and LDS
        # writes have no destination: all their operands are read)
        reads = args if op.startswith(("global_store", "buffer_store", "flat_store", "ds_write", "ds_store",
                                       "global_atomic", "v_cmp")) else args[1:]
        for a in reads:
            sp = _reg_span(a)
            hit = sp and next((r for r in results if r[1][0] == sp[0] and r[1][1] <= sp[2] and sp[1] <= r[1][2]), None)
            if hit:
                problems.append("line %d (%s): read of an MFMA result %d wait state(s) after the MFMA: %s"
                                % (ln, kernel, hit[0], text))
                break
        dst = None
        if op.startswith("v_") and not op.startswith(("v_cmp", "v_readlane", "v_readfirstlane")) and args:
            sp = _reg_span(args[0])
            if sp and (sp[0] == "v" or op.startswith("v_accvgpr_write")):
                dst = sp
        history.append((1, dst))
        age(1)
        if len(history) > 8:
            del history[0]
    return problems


def _counts_transfers(symbol: str) -> bool:
    """Whether a kernel waits for its transfers to LDS by the number of loads that it has requested behind them."""
    return re.match(r"_ZN5graft\d+tree_attn_parts_kernelI", symbol) is not None


def _is_transfer(op: str, text: str) -> bool:
    return "_lds_" in op or op.startswith("buffer_load") and text.endswith(" lds")


def _control_flow(body: str, first_line: int):
    """Instructions of a kernel as (line, opcode, text, in inline assembly), and of each the indices of those that may follow it."""
    code, label_at, in_asm = [], {}, False         # label -> index of the next instruction
    for ln, raw in enumerate(body.split("\n"), first_line):
        in_asm = ("ASMSTART" in raw or in_asm) and "ASMEND" not in raw
        text = raw.split(";")[0].strip()
        if re.match(r"\.\w+:", text):
            label_at[text.split(":")[0]] = len(code)
        elif text and not text.startswith("."):
            code.append((ln, text.split()[0], text, in_asm))
    after = []
    for i, (_, op, text, _) in enumerate(code):
        jump = [label_at[text.split()[1]]] if op.startswith(("s_branch", "s_cbranch")) else []
        after.append([] if op == "s_endpgm" else jump if op == "s_branch" else jump + [i + 1])
    return code, after


def _check_transfers(asm_text: str):
    """Transfers from memory straight to LDS are inline assembly, and nothing but the kernels' own s_waitcnt waits for them.
    Behind the last MFMA wavefronts exchange results in the LDS that keys and queries came to.  On every path of the
    control-flow graph, whatever the lengths, the transfers of all wavefronts must have landed there before LDS is
    written, which takes a vmcnt(0) and a barrier behind it."""
    LANDED, MINE_LANDED, IN_FLIGHT = 0, 1, 2
    problems = []
    for body in re.finditer(r"^(_Z\w+):[^\n]*\n(.*?)^\.Lfunc_end", asm_text, re.M | re.S):
        counts = _counts_transfers(body.group(1))
        if not counts and not _managed_accvgprs(body.group(1)):
            continue
        code, after = _control_flow(body.group(2), asm_text.count("\n", 0, body.start(2)) + 1)
        before = [[] for _ in code]
        for i, targets in enumerate(after):
            for t in targets:
                before[t].append(i)
        ahead = {i for i, c in enumerate(code) if c[1].startswith("v_mfma")}        # an MFMA may follow
        todo = list(ahead)
        while todo:
            for i in before[todo.pop()]:
                if i not in ahead:
                    ahead.add(i)
                    todo.append(i)
        if counts:
            problems += _check_counted_waits(body.group(1), code, after, set(range(len(code))) - ahead)
            continue
        state = [None] * len(code)                 # of the transfers in front of an instruction, the worst of all paths
        state[0], todo = LANDED, [0]
        while todo:
            i = todo.pop()
            op, text, s = code[i][1], code[i][2], state[i]
            if _is_transfer(op, text):
                s = IN_FLIGHT
            elif op == "s_waitcnt" and "vmcnt(0)" in text:
                s = min(s, MINE_LANDED)
            elif op == "s_barrier" and s == MINE_LANDED:
                s = LANDED
            for t in after[i]:
                if state[t] is None or state[t] < s:
                    state[t] = s
                    todo.append(t)
        for i, (ln, op, text, _) in enumerate(code):
            if op.startswith("ds_write") and i not in ahead and state[i]:
                problems.append("line %d (%s): transfers to LDS may be in flight: %s" % (ln, body.group(1), text))
    return problems


def _span(token: str):
    """Scalar registers of an operand: 's7' -> (7, 7), 's[2:3]' -> (2, 3), vcc -> (-1, -1), none -> None."""
    m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", token)
    if m:
        return int(m.group(1) or m.group(2)), int(m.group(1) or m.group(3))
    return (-1, -1) if token.startswith("vcc") else None


def _written_scalars(op: str, args):
    """Spans of the scalar registers that an instruction may write."""
    if op.startswith(("s_cmp", "s_bitcmp", "s_cbranch", "s_branch", "s_waitcnt", "s_barrier", "s_nop", "s_endpgm", "s_sleep", "s_setprio",
                      "ds_", "global_", "buffer_", "flat_", "scratch_")):
        return []
    spans = [x for x in map(_span, args[:2 if op.startswith("v_") else 1]) if x]
    return spans + ([(-1, -1)] if op.startswith("v_cmp") and op.endswith("e32") else [])


class _Facts:
    """What a path knows of scalar conditions.  A condition is (relation, whether it holds where the relation does); relations are of
    registers as they are: a write of one ends what is known of it.  Few are kept, the newest."""
    __slots__ = ("vcc", "scc", "pairs", "known")

    def __init__(self, vcc=None, scc=None, pairs=(), known=()):
        self.vcc, self.scc, self.pairs, self.known = vcc, scc, pairs, known

    def key(self):
        return self.vcc, self.scc, self.pairs, self.known

    def after(self, op: str, args):
        vcc, scc, pairs, known = self.key()
        if op.startswith("s_") and not op.startswith(("s_cselect", "s_mov", "s_cbranch", "s_waitcnt", "s_nop", "s_load", "s_barrier", "s_mul_i32")):
            scc = None                             # (most of them write it)
        new_pair, new_vcc = None, None
        if op == "s_cselect_b64" and self.scc and args[1:] in (["-1", "0"], ["0", "-1"]):
            new_pair = self.scc[0], self.scc[1] == (args[1] == "-1")
        if op in ("s_and_b64", "s_andn2_b64") and args[:2] == ["vcc", "exec"]:
            of = dict(pairs).get(_span(args[2]), (("bits", args[2]), True))
            new_vcc = of[0], of[1] == (op == "s_and_b64")
        for lo, hi in _written_scalars(op, args):
            hit = lambda c: any(x and x[0] <= hi and lo <= x[1] for x in map(_span, c[0][1:]))
            pairs = tuple((r, c) for r, c in pairs if (hi < r[0] or r[1] < lo) and not hit(c))
            known = tuple(c for c in known if not hit(c))
            vcc = None if lo < 0 or vcc and hit(vcc) else vcc
            scc = None if scc and hit(scc) else scc
        if new_pair:
            pairs = (pairs + ((_span(args[0]), new_pair),))[-3:]
        vcc = new_vcc or vcc
        m = re.fullmatch(r"s_cmp_(lt|ge|gt|le|eq|lg)_([iu]\d+)", op)
        if m:
            x, y = args if m.group(1) in ("lt", "ge", "eq", "lg") else args[::-1]
            scc = ("eq" if m.group(1) in ("eq", "lg") else "lt_" + m.group(2), x, y), m.group(1) in ("lt", "gt", "eq")
        return _Facts(vcc, scc, pairs, known)

    def branch(self, op: str, taken: bool):
        """The facts behind a branch, or None where what is known rules it out."""
        cond = self.vcc if "vcc" in op else self.scc if "scc" in op else None
        if cond is None:
            return self
        holds = (taken == op.endswith(("nz", "scc1"))) == cond[1]
        if (cond[0], not holds) in self.known:
            return None
        return _Facts(self.vcc, self.scc, self.pairs, (tuple(c for c in self.known if c[0] != cond[0]) + ((cond[0], holds),))[-3:])


def _check_counted_waits(kernel: str, code, after, behind_mfma):
    """The kernel's own s_waitcnt vmcnt(N) stand for "the transfers have landed, the loads behind them may be on their way": on every
    path at least N loads or stores must have been requested behind the last transfer, or a shorter wait must stand in between.  And where
    LDS is written behind the last MFMA, all wavefronts' transfers must have landed: a barrier behind such a wait.
    Paths are those that scalar conditions allow: the next tile's keys and, behind the products, its values are requested by one."""
    LANDED = 1 << 10
    # of every instruction: facts -> (requests behind the last transfer, whether a barrier has followed its landing), the worst of
    # all paths that arrive with them
    states, start = [{} for _ in code], _Facts()
    states[0][start.key()] = (LANDED, True)
    todo, problems, waits = [(0, start)], {}, 0
    while todo:
        i, facts = todo.pop()
        ln, op, text, in_asm = code[i]
        count, synced = states[i][facts.key()]
        wait = re.search(r"vmcnt\((\d+)\)", text) if op == "s_waitcnt" else None
        if wait and in_asm:
            waits += 1
            if count < int(wait.group(1)):
                problems[i] = "only %d requests behind the last transfer" % count
        if op.startswith("ds_write") and i in behind_mfma and not synced:
            problems[i] = "transfers to LDS may be in flight"
        if _is_transfer(op, text):
            count, synced = 0, False
        elif op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            count = min(count + 1, LANDED)
        elif wait and count >= int(wait.group(1)):
            count = LANDED
        elif op == "s_barrier" and count == LANDED:
            synced = True
        facts = facts.after(op, text.replace(",", " ").split()[1:])
        for n, t in enumerate(after[i]):
            there = facts.branch(op, n == 0) if len(after[i]) == 2 else facts            # (the first one is where a branch goes)
            if there is None:
                continue
            old = states[t].get(there.key(), (LANDED + 1, True))
            worst = (min(old[0], count), old[1] and synced)
            if worst != old:
                states[t][there.key()] = worst
                todo.append((t, there))
    if not waits and any(_is_transfer(op, text) for _, op, text, _ in code):
        return ["%s: no wait for its transfers found" % kernel]
    return ["line %d (%s): %s: %s" % (code[i][0], kernel, what, code[i][2]) for i, what in sorted(problems.items())]


def _check_and_clean(directory: str, what: str):
    for src in HAND_SCHEDULED:
        with open(_asm_of(src, directory)) as f:
            problems = check_attention_asm(f.read())
        if problems:
            raise RuntimeError("%s%s: the generated assembly breaks a rule of the hand-scheduled kernels:\n  "
                               % (src, what) + "\n  ".join(problems[:20]))
    for name in os.listdir(directory):           # the other intermediate files are not needed
        if name.startswith("tree_attn") and not name.endswith((".o", "gfx950.s")) or name.endswith(".hipfb"):
            os.remove(os.path.join(directory, name))


def _link(objects, lib: str) -> str:
    tmp = lib + ".tmp%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", tmp]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, lib)
    return lib


def build_native() -> str:
    """_native.so: plain C++ against the headers of PyTorch and Python.  It resolves libgraft.so at run
    time (bind()), and PyTorch's libraries are the ones `import torch` has loaded."""
    import torch
    base = os.path.dirname(os.path.abspath(torch.__file__))
    inc, libs = os.path.join(base, "include"), os.path.join(base, "lib")
    tmp = NATIVE + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-sign-compare", "-I", INCLUDE,
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"],
           "-isystem", "/opt/rocm/include",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L", libs, "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10", "-ldl"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("the native binding does not build:\n" + r.stdout)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every HIP source and link libgraft.so next to the package, and build _native.so.  Always recompiles."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(9, len(SOURCES) + 1)) as ex:
        native = ex.submit(build_native)
        results = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        native.result()
    if verbose:
        for _, w in results:
            if w:
                print(w)
    _check_and_clean(OBJ_DIR, "")
    return _link([o for o, _ in results], LIB)


def build_timing(verbose: bool = False) -> str:
    """libgraft_timing.so: the library with the attention kernel compiled with -DGRAFT_ATTN_STAMPS
    (time stamps per workgroup, read by `python -m paper_2605_20104_amd.timing`).  The other
    objects are those of the last build(); the stamped kernels pass the same assembly check."""
    others = [os.path.join(OBJ_DIR, os.path.splitext(s)[0] + ".o") for s in SOURCES if s not in HAND_SCHEDULED]
    if not all(os.path.exists(o) for o in others):
        build(verbose)
    src_dir = os.path.join(OBJ_DIR, "timing")
    os.makedirs(src_dir, exist_ok=True)
    objects = [os.path.join(src_dir, os.path.splitext(s)[0] + ".o") for s in HAND_SCHEDULED]
    with ThreadPoolExecutor(max_workers=len(objects)) as ex:
        results = list(ex.map(lambda x: _compile_to(x[0], ["-DGRAFT_ATTN_STAMPS"], x[1]), zip(HAND_SCHEDULED, objects)))
    if verbose:
        for _, warn in results:
            if warn:
                print(warn)
    _check_and_clean(src_dir, " (timing build)")
    return _link([*objects, *others], LIB_TIMING)


if __name__ == "__main__":
    flags = [a for a in sys.argv[1:] if a != "--timing"]
    print(build(verbose=True, extra_flags=flags))
    if "--timing" in sys.argv[1:]:
        print(build_timing(verbose=True))
