"""The built kernels keep the distance that the hardware asks for between a matrix
product and the next instruction that touches its result.

On gfx950 eight wait states (one per instruction, n + 1 for s_nop n) have to lie
between v_mfma_f32_16x16x32_bf16 and a vector, LDS or memory instruction that reads or
overwrites the registers it writes; nothing interlocks them.  The compiler keeps to
that inside a block, but over an edge it can count a branch that is not on the path
(mfma_settle in gpa_device.h).  This walks every path behind every product in the
disassembly of the library."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

import paper_2609_34272_amd as gpa

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT = 8


def _regs(operands):
    out = set()
    for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", operands):
        if m[1]:
            out |= {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
        else:
            out.add((m[4], int(m[5])))
    return out


def _kernels(text):
    """{kernel: (instructions as (opcode, operands), {label: index})}"""
    kernels, ins, labels = {}, None, None
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        m = re.match(r"[0-9a-f]+ <(\w+)>:$", line)
        if m and re.fullmatch(r"L\d+", m[1]):
            labels[m[1]] = len(ins)
        elif m:
            ins, labels = [], {}
            kernels[m[1]] = (ins, labels)
        elif line and ins is not None:
            op, _, args = line.partition(" ")
            ins.append((op, args))
    return kernels


def early_accesses(ins, labels):
    """(wait states, product, instruction) for each access that comes too early."""
    found = []
    for i, (op, args) in enumerate(ins):
        if not op.startswith("v_mfma"):
            continue
        dst = _regs(args.split(",")[0])
        seen, todo = {}, [(i + 1, 0)]
        while todo:
            j, waited = todo.pop()
            while j < len(ins) and waited < WAIT and seen.get(j, WAIT) > waited:
                seen[j] = waited
                op2, args2 = ins[j]
                if op2.startswith("v_mfma"):
                    if _regs(args2.split(",")[0]) & dst:
                        break  # from here on it is that product's result
                elif not op2.startswith("s_") and _regs(args2) & dst:
                    found.append((waited, f"{op} {args}", f"{op2} {args2}"))
                    break
                waited += int(args2) + 1 if op2 == "s_nop" else 1
                if op2.startswith("s_cbranch"):
                    todo.append((labels[args2.strip()], waited))
                elif op2 == "s_branch":
                    j = labels[args2.strip()]
                    continue
                elif op2 == "s_endpgm":
                    break
                j += 1
    return found


def test_the_walk_finds_early_accesses():
    """On hand-made code: in line, over both ends of a branch, and past a loop edge."""
    product = ("v_mfma_f32_16x16x32_bf16", "v[0:3], v[8:11], v[12:15], v[0:3]")
    use, other, nop = ("v_mov_b32_e32", "v20, v2"), ("v_mov_b32_e32", "v20, v21"), ("s_nop", "6")
    assert early_accesses([product, nop, use], {}) == [(7, " ".join(product), " ".join(use))]
    assert not early_accesses([product, nop, other, use], {})
    assert early_accesses([product, ("v_mov_b32_e32", "v3, 0")], {})
    code = [use, product, ("s_nop", "4"), ("s_cbranch_scc1", "L0"), ("s_nop", "1"), use]
    assert [w for w, *_ in early_accesses(code, {"L0": 0})] == [6]
    assert [w for w, *_ in early_accesses(code[:4] + [use], {"L0": 4})] == [6]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_result_of_a_product_is_touched_too_early(tmp_path):
    gpa.lib()
    shutil.copy(gpa.LIB_PATH, tmp_path / "libgpa.so")
    subprocess.run([OBJDUMP, "--offloading", "libgpa.so"], cwd=tmp_path, check=True, capture_output=True)
    products = 0
    for f in sorted(tmp_path.glob("*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", str(f)],
                              check=True, capture_output=True, text=True).stdout
        for kernel, (ins, labels) in _kernels(text).items():
            ops = {op for op, _ in ins if op.startswith("v_mfma")}
            assert ops <= {"v_mfma_f32_16x16x32_bf16"}, (kernel, ops)  # the wait is this one's
            products += sum(op.startswith("v_mfma") for op, _ in ins)
            early = early_accesses(ins, labels)
            assert not early, (kernel, min(early))
    assert products > 1000
