"""Waits between matrix instructions and what reads or overwrites their results, in the machine code
of the built library.  The compiler inserts these waits, but it counts them before the last changes
of branches, and where blocks join it can miss the shorter way; this walks every way through
every kernel.  States needed: what the compiler itself keeps on gfx950, from the passes of an
instruction: passes + 4 for the bf16 and fp16 products (8 passes, 4 for 16x16x32), passes + 2 for the fp32 ones (8)."""
import glob
import os
import re
import subprocess

import pytest

from paper_2310_01655_amd import build as lib_build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STATES = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x16_f16": 12, "v_mfma_f32_16x16x4_f32": 10,
          "v_mfma_f32_16x16x32_bf16": 8}
STORES = ("ds_write", "ds_bpermute", "global_store", "buffer_store", "scratch_store", "flat_store", "global_atomic")


def registers(operand):
    m = re.match(r"-?\|?([va])\[(\d+):(\d+)\]", operand.strip())
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"-?\|?([va])(\d+)\b", operand.strip())
    return {(m[1], int(m[2]))} if m else set()


def split_operands(text):
    return re.split(r",(?![^\[]*\])", text) if text else []


def parse(text):
    """{function: [(opcode, operands, reads, writes)]}; labels are ("label", name, ...)."""
    functions, code = {}, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(.+)>:", line)
        if m and not re.fullmatch(r"L\d+", m[1]):
            code = functions.setdefault(m[1], [])
        elif m:
            code.append(("label", m[1], set(), set()))
        elif line.startswith("\t") and code is not None:
            op, _, rest = line.split("//")[0].strip().partition(" ")
            ops = split_operands(rest)
            if op.startswith(STORES):
                reads, writes = set().union(*map(registers, ops)), set()
                if op.startswith("ds_bpermute"):
                    reads, writes = set().union(*map(registers, ops[1:])), registers(ops[0])
            else:
                reads = set().union(*map(registers, ops[1:])) if ops else set()
                writes = registers(ops[0]) if ops else set()
                if "fmac" in op or "dot2c" in op or "swap" in op:
                    reads |= writes
                if "swap" in op:
                    writes |= registers(ops[1])
            code.append((op, rest, reads, writes))
    return functions


def early_accesses(name, code):
    labels = {c[1]: i for i, c in enumerate(code) if c[0] == "label"}
    found = []
    for start, (op, rest, _, result) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        need, seen = STATES[op], {}
        ways = [(start + 1, 0, frozenset(result), False)]
        while ways:
            at, waited, pending, idle = ways.pop()       # idle: no lane is active, only matrix instructions act
            while at < len(code) and waited < need and pending:
                if (at, pending, idle) in seen and seen[at, pending, idle] <= waited:
                    break
                seen[at, pending, idle] = waited
                op2, rest2, reads, writes = code[at]
                if op2 == "s_endpgm":
                    break
                if op2 == "s_nop":
                    waited += int(rest2, 0)
                if op2 == "s_branch":
                    at, waited = labels[rest2.split()[0]], waited + 1
                    continue
                if op2.startswith("s_cbranch"):
                    ways.append((labels[rest2.split()[0]], waited + 1, pending, idle or op2 == "s_cbranch_execz"))
                if "saveexec" in op2 or rest2.startswith("exec"):
                    idle = False
                if op2.startswith("v_mfma"):
                    # sums may be continued in the same registers: the next product waits by itself
                    a, b, c = (registers(x) for x in split_operands(rest2)[1:4])
                    reads, writes = a | b | (c if c != result else set()), writes if c != result else set()
                    if c == result:
                        pending = pending - result       # (the later product is looked at on its own)
                elif idle:
                    reads, writes = set(), set()
                if (reads | writes) & pending:
                    found.append("%s: %s at %d, %s %s at %d after %d of %d" % (name, op, start, op2, rest2, at, waited, need))
                    break
                if op2 != "label":
                    waited += 1
                at += 1
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_results_of_matrix_instructions_are_waited_for(tmp_path):
    if not os.path.exists(lib_build.LIB):
        lib_build.build()
    copy = tmp_path / "lib.so"
    copy.symlink_to(lib_build.LIB)
    subprocess.run([OBJDUMP, "--offloading", str(copy)], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    objects = sorted(glob.glob(str(tmp_path / "*gfx950")))
    assert objects
    products, found = 0, []
    for path in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", path], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        for name, code in parse(text).items():
            products += sum(c[0].startswith("v_mfma") for c in code)
            found += early_accesses(name, code)
    assert products > 1000
    assert not found, "%d accesses too early:\n%s" % (len(found), "\n".join(found[:40]))
