"""The 256x256 tile of the prefill GEMM issues its matrix instructions as inline assembly, in place in the accumulator
registers.  The compiler's hazard recogniser does not look into assembly, so the wait states between such an
instruction and whatever else touches its registers are the source's to keep - and whether anything else does is up to
the register allocator.  This reads the assembly that the present compiler makes of the kernel and checks every path."""
import os
import re
import subprocess

import pytest

from paper_2401_09670_amd import build

AFTER = 8    # wait states after a four-pass matrix instruction before its result is read, moved or overwritten
BEFORE = 2   # between a vector instruction's result and a matrix instruction that reads it


class Instr:
    def __init__(self, text):
        self.text = text
        self.op, _, rest = text.partition(" ")
        self.matrix = self.op.startswith("v_mfma")
        self.operands = [_registers(o) for o in rest.split(",")] if rest else []
        self.touched = set().union(*self.operands) if self.operands else set()
        # s_nop n waits n + 1 states, everything else at least one
        self.states = int(rest, 0) + 1 if self.op == "s_nop" else 1
        target = re.match(r"s_c?branch\w* (\.L\w+)", text)
        self.target = target.group(1) if target else None
        self.falls_through = self.op not in ("s_branch", "s_endpgm", "s_setpc_b64")


def _registers(operand):
    regs = set()
    for kind, first, last, single in re.findall(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)", operand):
        lo, hi = (int(first), int(last)) if first else (int(single), int(single))
        regs.update((kind, r) for r in range(lo, hi + 1))
    return regs


def parse(lines):
    """Instructions of one function, and the index each label stands for."""
    code, labels = [], {}
    for line in lines:
        text = line.split(";")[0].strip()
        label = re.match(r"(\.L\w+):", text)
        if label:
            labels[label.group(1)] = len(code)
        elif text and not text.startswith("."):
            code.append(Instr(text.replace("\t", " ")))
    return code, labels


def _walk(code, labels, start, states):
    """Instructions that may be issued less than `states` wait states after number `start`."""
    seen, todo = {}, [(start, -1)]
    while todo:
        at, waited = todo.pop()
        if at != start or waited >= 0:
            if waited >= states or seen.get(at, states) <= waited:
                continue
            seen[at] = waited
            yield code[at]
        after = waited + code[at].states if at != start or waited >= 0 else 0
        if code[at].falls_through and at + 1 < len(code):
            todo.append((at + 1, after))
        if code[at].target in labels:
            todo.append((labels[code[at].target], after))


def hazards(code, labels):
    found = []
    for i, ins in enumerate(code):
        if ins.matrix:
            result = ins.operands[0]
            if ins.operands[3] != result:
                found.append(f"not in place: {ins.text}")
            for later in _walk(code, labels, i, AFTER):
                if later.matrix:
                    # accumulating on is what the hardware forwards; anything else of the result is not there yet
                    if (later.operands[1] | later.operands[2]) & result or \
                            (later.operands[0] & result and later.operands[0] != result):
                        found.append(f"{ins.text} -> {later.text}")
                elif later.touched & result:
                    found.append(f"{ins.text} -> {later.text}")
        elif ins.op.startswith("v_") and ins.operands:
            for later in _walk(code, labels, i, BEFORE):
                if later.matrix and later.touched & ins.operands[0]:
                    found.append(f"{ins.text} -> {later.text}")
    return found


def test_the_check_sees_what_it_is_for():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], a[0:3]"
    other = mfma.replace("a[0:3]", "a[4:7]")
    assert not hazards(*parse([mfma, other, mfma, "s_nop 6", "v_accvgpr_read_b32 v0, a4", "v_accvgpr_read_b32 v1, a3"]))
    assert hazards(*parse([mfma, "s_nop 6", "v_accvgpr_read_b32 v1, a3"]))
    assert hazards(*parse([mfma, "s_cbranch_scc0 .LBB0_1", "s_nop 7", ".LBB0_1:", "v_accvgpr_read_b32 v1, a3"]))
    assert hazards(*parse([".LBB0_1:", "v_accvgpr_write_b32 a1, v1", "s_nop 2", mfma, "s_nop 3", "s_branch .LBB0_1"]))
    assert hazards(*parse(["v_accvgpr_write_b32 a0, 0", "s_nop 0", mfma]))
    assert hazards(*parse(["v_mov_b32_e32 v9, v20", "s_mov_b32 s0, 0", mfma]))
    assert not hazards(*parse(["v_mov_b32_e32 v9, v20", "s_nop 1", mfma]))
    assert hazards(*parse([mfma, "v_mfma_f32_16x16x32_bf16 a[4:7], a[0:3], v[12:15], a[4:7]"]))
    assert hazards(*parse([mfma.replace(" a[0:3],", " a[4:7],", 1)]))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = os.path.join(tmp_path_factory.mktemp("asm"), "gemm.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    functions, name = {}, None
    for line in open(out):
        begin = re.match(r"(_Z\w*gemm_dl_kernelILi256ELi256E\w*):", line)
        if begin:
            name = begin.group(1)
            functions[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            functions[name].append(line)
    return {n: parse(lines) for n, lines in functions.items()}


def test_big_tile_kernels_keep_their_wait_states(kernels):
    assert len(kernels) >= 2                                  # plain and split-K at least
    for name, (code, labels) in kernels.items():
        assert sum(i.matrix for i in code) >= 2 * 128, name   # the loop's k-tile and the last one
        assert not hazards(code, labels), name


def test_big_tile_main_loop_moves_no_accumulator(kernels):
    """128 matrix instructions per k-tile and no move: what the 256x256 tile's speed rests on."""
    for name, (code, labels) in kernels.items():
        loops = [code[labels[c.target]:i + 1] for i, c in enumerate(code) if c.target in labels and labels[c.target] <= i]
        loops = [body for body in loops if any(c.matrix for c in body)]
        assert len(loops) == 1 and sum(c.matrix for c in loops[0]) == 128, name
        moves = [c.text for c in loops[0] if not c.matrix and any(kind == "a" for kind, _ in c.touched)]
        assert not moves, (name, moves[:4])
