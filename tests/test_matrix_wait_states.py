"""Wait states around matrix instructions written as inline assembly.

The compiler does not know such an instruction as one of the matrix pipe and places no wait states for it, so the sources
place them: two between a vector instruction that writes one of its operands and it, eighteen between it and whatever reads
or overwrites its result.  Whether they stand where they have to is decided by the order that the compiler gives the other
instructions; this test follows every path through the compiled kernels (built here from source, no GPU needed) and counts.
`s_nop n` is n + 1 states.  In front of a matrix instruction every other instruction is one, the least that it can take.
Behind one only `s_nop` counts: what else happens to stand there, another version of the compiler puts elsewhere."""

import glob
import os
import re
import subprocess

import pytest

from paper_2410_05265_amd import build

SOURCES = [os.path.basename(s) for s in build.sources() if "asm volatile(\"v_mfma" in open(s).read()]
AFTER_RESULT, AFTER_WRITE = 18, 2
REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")
# (vector stores and LDS writes write no register)
NO_RESULT = ("global_store", "flat_store", "buffer_store", "scratch_store", "ds_write", "global_load_lds", "v_cmp", "v_readfirstlane", "v_readlane")


def registers(text):
    out = set()
    for kind, one, lo, hi in REG.findall(text):
        first, last = (int(one), int(one)) if one else (int(lo), int(hi))
        out.update((kind, i) for i in range(first, last + 1))
    return frozenset(out)


class Instruction:
    """What an instruction does to the registers, in the terms of the rules above."""

    def __init__(self, line, in_asm):
        self.line, self.in_asm = line, in_asm
        op, _, rest = line.partition(" ")
        operands = [registers(o) for o in re.split(r",(?![^\[]*\])", rest)] if rest else []
        self.wait = op == "s_nop"
        self.states = int(rest) + 1 if self.wait else 1
        self.matrix = in_asm and op.startswith("v_mfma")
        self.result = operands[0] if self.matrix else frozenset()
        self.operands = operands[1] | operands[2] if self.matrix else frozenset()
        self.touched = frozenset().union(*operands) if operands and not self.matrix else frozenset()
        writes = op.startswith("v_") and not op.startswith(NO_RESULT) and operands and not self.matrix
        self.written = operands[0] | (operands[1] if writes and "swap" in op else frozenset()) if writes else frozenset()
        self.target = rest.strip() if op.startswith(("s_cbranch", "s_branch")) else None
        self.ends = op in ("s_branch", "s_endpgm", "s_setpc_b64")


def functions(asm):
    """name -> (list of blocks, label -> index of a block); a block is a list of instructions."""
    out, name, blocks, labels, in_asm = {}, None, None, None, False
    for raw in asm.splitlines():
        line = raw.split("; ")[0].split("//")[0].strip() if not raw.strip().startswith(";") else raw.strip()
        if m := re.match(r"^(_Z\w+|k_\w+):", raw):
            name, blocks, labels = m.group(1), [[]], {}
            out[name] = (blocks, labels)
        elif name is None:
            continue
        elif raw.startswith(".Lfunc_end"):
            name = None
        elif m := re.match(r"^(\.LBB\w+):", raw):
            blocks.append([])
            labels[m.group(1)] = len(blocks) - 1
        elif line.startswith(";"):
            in_asm = line.startswith(";APP") or line.startswith(";;#ASMSTART") or (in_asm and not line.startswith((";NO_APP", ";;#ASMEND")))
        elif line and not line.startswith("."):
            ins = Instruction(line, in_asm)
            blocks[-1].append(ins)
            if ins.target:
                blocks.append([])          # (what follows a branch is a block of its own)
    return out


def step(pending, ins, report):
    """pending: (register, rule) -> states that still have to pass.  Returns it behind `ins`."""
    if pending:
        for (reg, rule), left in pending.items():
            if rule == "result":
                wrong = reg in ins.touched or reg in ins.operands
            else:
                wrong = reg in ins.operands or reg in ins.result
            if wrong and left > 0:
                report.append("%s: %s%d is %s %d states too early" % (ins.line, *reg, rule, left))
        passed = {"result": ins.states if ins.wait else 0, "operand": ins.states}
        pending = {k: left - passed[k[1]] for k, left in pending.items() if left > passed[k[1]]}
    for reg in ins.result:
        pending[reg, "result"] = AFTER_RESULT
    for reg in ins.written:
        pending[reg, "operand"] = AFTER_WRITE
    return pending


def violations(blocks, labels, step=step):
    report, entry, todo = [], {0: {}}, [0]
    while todo:
        at = todo.pop()
        pending = dict(entry[at])
        follow = [at + 1]
        for ins in blocks[at]:
            pending = step(pending, ins, report)
            if ins.target and ins.target in labels:
                follow.append(labels[ins.target])
            if ins.ends:
                follow.remove(at + 1)
        for nxt in follow:
            if nxt >= len(blocks):
                continue
            known = entry.get(nxt)
            merged = dict(known or {})
            for k, left in pending.items():
                merged[k] = max(left, merged.get(k, 0))
            if known is None or merged != known:
                entry[nxt] = merged
                todo.append(nxt)
    return report


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not installed")
    folder = tmp_path_factory.mktemp("asm")
    procs = [(s, subprocess.Popen([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, s), "-o", str(folder / s)],
                                  stderr=subprocess.PIPE, text=True)) for s in SOURCES]
    out = {}
    for s, pr in procs:
        _, err = pr.communicate()
        assert pr.returncode == 0, err[-4000:]
        out[s] = (folder / s).read_text()
    return out


@pytest.mark.parametrize("source", SOURCES)
def test_results_and_operands_are_waited_for(compiled, source):
    found = 0
    for name, (blocks, labels) in functions(compiled[source]).items():
        if not any(i.matrix for b in blocks for i in b):
            continue
        found += 1
        bad = violations(blocks, labels)
        assert not bad, "%s: %d, first %s" % (name, len(bad), bad[:3])
    assert found                                    # (the parser still finds the instructions it is there for)


@pytest.mark.parametrize("source", SOURCES)
def test_nothing_is_spilled(compiled, source):
    """Memory operations of a wavefront retire in order: the reload of a spilled register behind direct loads to LDS waits for
    all of them, and with that for the operands of a tile whose loads were issued early to overlap the last one's epilogue."""
    sizes = [int(n) for n in re.findall(r"\.private_segment_fixed_size: (\d+)", compiled[source])]
    assert sizes and not any(sizes), sizes


@pytest.mark.parametrize("lines,bad", [
    (["v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]", "v_accvgpr_read_b32 v9, a3"], 1),
    (["v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 15", "s_nop 1", "v_accvgpr_read_b32 v9, a3"], 0),
    (["v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 15", "s_nop 0", "v_accvgpr_read_b32 v9, a3"], 1),
    (["v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]"] + ["v_add_u32_e32 v9, v9, v9"] * 40 + ["v_accvgpr_read_b32 v9, a3"], 1),
    (["v_mov_b32_e32 v5, 0", "v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]"], 1),
    (["v_mov_b32_e32 v5, 0", "s_nop 1", "v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]"], 0),
    (["v_accvgpr_write_b32 a1, v9", "s_nop 0", "v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]"], 1),
    (["v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]", "v_mfma_x a[0:3], v[0:3], v[4:7], a[0:3]"], 0)])
def test_the_count_itself(lines, bad):
    body = "".join("\t;;#ASMSTART\n\t%s\n\t;;#ASMEND\n" % t if "mfma" in t else "\t%s\n" % t for t in lines)
    blocks, labels = functions("_Zk:\n%s\ts_endpgm\n.Lfunc_end0:\n" % body)["_Zk"]
    assert (len(violations(blocks, labels)) > 0) == bool(bad)
