"""Waits between matrix instructions and the vector instructions around them, in the code as built.

Some kernels multiply accumulators inside assembly, where the compiler does not count these waits.  On gfx950 a vector
instruction may touch the result of a 16x16x32 matrix instruction eight instructions after it (s_nop N counts as N + 1) and
that of a 32x32x16 one after twelve, and a matrix instruction may read a register two instructions after a vector
instruction has written it: what the compiler itself puts between them."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2311_11822_amd", "libdp_bk.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
RESULT_WAIT = {"16x16x32": 8, "32x32x16": 12}
OPERAND_WAIT = 2
ENDS = ("s_branch", "s_endpgm", "s_setpc_b64")           # nothing runs on behind these
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def registers(operand):
    regs = set()
    for kind, one, lo, hi in REG.findall(operand):
        regs.update((kind, r) for r in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1)))
    return regs


class Instruction:
    def __init__(self, text, address):
        self.text, self.address = text, address
        self.name, _, rest = text.partition(" ")
        self.operands = [o.strip() for o in re.split(r",(?![^\[]*\])", rest)]
        self.matrix = next((w for shape, w in RESULT_WAIT.items() if "v_mfma" in self.name and shape in self.name), 0)
        self.vector = self.name.startswith("v_") and "mfma" not in self.name
        self.states = int(rest, 0) + 1 if self.name == "s_nop" else 1


def too_close(code, target):
    """Pairs (earlier, later) of a run of instructions, the later one from index `target` on, that are closer than allowed."""
    found = []
    for j in range(target, len(code)):
        later = code[j]
        if later.matrix:
            reads = set().union(*(registers(o) for o in later.operands[1:]))
        elif later.vector:
            reads = set().union(*(registers(o) for o in later.operands))
        else:
            continue
        states = 0
        for i in range(j - 1, -1, -1):
            earlier = code[i]
            if states >= max(RESULT_WAIT.values()):
                break
            if later.matrix and earlier.vector and states < OPERAND_WAIT and registers(earlier.operands[0]) & reads:
                found.append((earlier.text, later.text, states))
            if later.vector and earlier.matrix and states < earlier.matrix and registers(earlier.operands[0]) & reads:
                found.append((earlier.text, later.text, states))
            states += earlier.states
    return found


def check(lines):
    """Straight runs, and every jump together with what comes before it and what it leads to."""
    code, starts = [], {}
    for line in lines:
        m = re.match(r"\s+([a-z]\w+.*?)\s*//\s*([0-9A-F]+):", line)
        if m:
            code.append(Instruction(m.group(1), int(m.group(2), 16)))
            starts[code[-1].address] = len(code) - 1
    found, reach, begin = [], max(RESULT_WAIT.values()), 0
    for i, ins in enumerate(code):
        if ins.name == "s_branch" or ins.name.startswith("s_cbranch"):
            offset = int(ins.operands[0], 0)
            to = starts[ins.address + 4 + 4 * (offset - (1 << 16) if offset >= 1 << 15 else offset)]
            before, after = code[max(begin, i - reach):i + 1], code[to:to + reach]
            last = next((k for k, x in enumerate(after) if x.name in ENDS), len(after))
            found += too_close(before + after[:last], len(before))
        if ins.name in ENDS or i == len(code) - 1:
            found += too_close(code[begin:i + 1], 0)
            begin = i + 1
    return found


def disassembly(library, folder):
    """Lines of each kernel of each code object in a library."""
    copy = os.path.join(str(folder), "library.so")
    shutil.copy(library, copy)
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, stdout=subprocess.DEVNULL)
    for name in sorted(os.listdir(str(folder))):
        if name.endswith("gfx950"):
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(str(folder), name)], check=True,
                                  capture_output=True, text=True).stdout
            for part in re.split(r"\n(?=[0-9a-f]+ <)", text)[1:]:
                lines = part.splitlines()
                yield lines[0].partition("<")[2].rstrip(">:"), lines[1:]


@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(LIB), reason="needs the built library and a disassembler")
def test_waits_of_matrix_instructions(tmp_path):
    kernels, faults = 0, []
    for name, lines in disassembly(LIB, tmp_path):
        kernels += 1
        faults += [(name, *f) for f in check(lines)]
    assert kernels > 50
    assert not faults, f"{len(faults)} pairs: " + "; ".join(map(str, faults[:8]))


# The gradient kernels store rows in three forms: old values added (cached), streaming and cached (64 x 64 tiles: the first two).  The
# compiler makes one cached form of the last two unless it is kept from it.
@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(LIB), reason="needs the built library and a disassembler")
def test_gradient_kernels_stream_and_do_not(tmp_path):
    kernels = 0
    for name, lines in disassembly(LIB, tmp_path):
        if re.search(r"clipped_grad_(big|blocks|mid|mid_blocks|tail)_kernel|grad_packed_kernel", name):
            stores = [line for line in lines if "global_store_dwordx4" in line]
            streaming = sum(bool(re.search(r"\bnt\b", line)) for line in stores)
            kernels += 1
            forms = 2 if "tail" in name else 3
            assert streaming > 0 and len(stores) == forms * streaming, (name, streaming, len(stores))
    assert kernels == 8 * 7 + 4


def test_the_check_finds_what_is_too_close():
    def run(*names):
        return check([f"\t{n} // {4 * i:012X}: " for i, n in enumerate(names)])
    matrix, nop = "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[4:7]", "s_nop 0"
    multiply = "v_mul_f32_e32 v7, s3, v7"
    assert run(multiply, nop, matrix) and not run(multiply, "s_nop 1", matrix)
    assert run(matrix, "s_nop 6", multiply) and not run(matrix, "s_nop 7", multiply)
    assert run(matrix.replace("16x16x32", "32x32x16"), "s_nop 10", multiply)
    assert not run(matrix, nop, "v_mul_f32_e32 v16, s3, v17") and not run(multiply, "s_endpgm", matrix)
    assert run(matrix, "s_nop 7", multiply, "s_cbranch_scc1 65532")               # back to the matrix instruction
    assert not run(matrix, "s_nop 7", multiply, nop, "s_cbranch_scc1 65531")
