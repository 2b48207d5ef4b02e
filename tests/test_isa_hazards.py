"""Wait states that the gfx950 ISA asks of the program, in the built library.

The compiler keeps them for its own instructions; an instruction inside an
inline-assembly block is the author's to space.  The library's device code
(compiled here from csrc/) is disassembled and, along every path of the
control flow, two rules are checked:
  * a vector-memory instruction reads an SGPR at the earliest five wait states
    after a vector instruction (v_readfirstlane, v_cmp ..) wrote it;
  * an LDS-DMA load comes at the earliest one wait state after a scalar write
    of M0, its LDS base.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_02963_amd import _build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VMEM = ("global_", "buffer_", "flat_", "scratch_")
INSTR = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]{12}): ([0-9A-F]{8})")


def _sgprs(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m[1])}
    return {operand} if operand in ("vcc", "m0") else set()


def _functions(text):
    """{name: [(address, opcode, operands, first word)]}"""
    out, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"^<(\S+)>:$", line) or re.match(r"^[0-9a-f]+ <(\S+)>:$", line)
        if m:
            cur = out.setdefault(m[1], [])
            continue
        m = INSTR.match(line)
        if m and cur is not None:
            cur.append((int(m[3], 16), m[1], [a.split()[0] for a in m[2].split(",") if a.split()], int(m[4], 16)))
    return out


def _written(op, args):
    """SGPRs that a vector instruction writes, and M0 by a scalar one."""
    if op.startswith("v_"):
        w = _sgprs(args[0]) if args else set()
        if op.startswith(("v_add_co", "v_sub_co", "v_addc", "v_subb", "v_mad_u64", "v_mad_i64", "v_div_scale")):
            w |= _sgprs(args[1])
        return w
    return {"m0"} if op.startswith("s_") and args and args[0] == "m0" else set()


def hazards(instrs):
    """(address, opcode, what) of every instruction that follows too closely on some path."""
    at = {a: i for i, (a, *_) in enumerate(instrs)}
    before = [[] for _ in instrs]
    for i, (a, op, _, word) in enumerate(instrs):
        if op.startswith(("s_branch", "s_cbranch")):
            imm = word & 0xFFFF
            j = at.get(a + 4 + 4 * (imm - 0x10000 if imm & 0x8000 else imm))
            if j is not None:
                before[j].append(i)
        if not op.startswith(("s_branch", "s_endpgm", "s_setpc")) and i + 1 < len(instrs):
            before[i + 1].append(i)
    found = []
    for i, (a, op, args, _) in enumerate(instrs):
        if not op.startswith(VMEM):
            continue
        rules = [(5, set().union(*(_sgprs(x) for x in args)) if args else set(), "SGPR")]
        if "_lds_" in op or "lds" in args:
            rules.append((1, {"m0"}, "M0"))
        for need, regs, what in rules:
            seen, todo = {}, [(j, 0) for j in before[i]]
            while todo and regs:
                j, d = todo.pop()
                if d >= need or seen.get(j, need) <= d:
                    continue
                seen[j] = d
                _, o, x, _ = instrs[j]
                if _written(o, x) & regs:
                    found.append((hex(a), op, f"{what} written {d} wait states before by {o}"))
                    break
                step = int(x[0], 0) + 1 if o == "s_nop" else 1
                todo += [(k, d + step) for k in before[j]]
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not found")
def test_inline_assembly_keeps_the_wait_states(tmp_path):
    so = shutil.copy(_build.LIBRARY, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", so], cwd=tmp_path, check=True, capture_output=True)
    images = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    dmas = 0
    for image in images:
        text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp_path, image)], check=True, capture_output=True, text=True).stdout
        for name, instrs in _functions(text).items():
            dmas += sum("_lds_" in op for _, op, _, _ in instrs)
            assert hazards(instrs) == [], name
    assert len(images) >= 4 and dmas > 100  # the kernels were read


def test_the_check_sees_a_close_write_on_a_branch():
    """Four wait states are too few, five are enough, a nop counts its own, and a taken branch is followed."""
    def listing(nop):
        lines = ["v_readfirstlane_b32 s4, v1", "s_mov_b32 m0, s9", f"s_nop {nop}", "s_branch 1", "s_endpgm",
                 "global_load_lds_dwordx4 v2, s[4:5]"]
        out, word = "<k>:\n", {"s_branch 1": 0xBF820001}
        for i, x in enumerate(lines):
            out += "\t%s // %012X: %08X\n" % (x, 4 * i, word.get(x, 0))
        return hazards(_functions(out)["k"])
    assert len(listing(1)) == 1 and "SGPR" in listing(1)[0][2]
    assert listing(2) == []
