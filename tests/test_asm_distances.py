"""Vector instructions in assembly statements next to matrix products.  The hardware does not hold an instruction back until what it
reads is there; the compiler places wait states for its own instructions, but does not look into assembly.  The compiled kernels are
searched for a statement that stands too close, along every path, loops included:

  * an instruction of a statement that touches a matrix product's result: twelve wait states behind it (as many as the compiler leaves
    for its own instructions behind the eight-pass products used here);
  * a matrix product that reads what a statement wrote: two behind it;
  * a reader of what a sub-dword operation wrote: one behind it;
  * a row operation (DPP) of a statement: two behind the vector instruction that wrote its operand.
"""
import os
import pathlib
import re
import shutil
import subprocess

import pytest

CSRC = pathlib.Path(__file__).parents[1] / "paper_2410_23918_amd" / "csrc"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
BEHIND_PRODUCT, BEFORE_PRODUCT, BEHIND_SUBDWORD, BEFORE_ROW = 12, 2, 1, 2


def registers(operand):
    """the vector registers (a: accumulation) that an operand names"""
    found = set()
    for kind, one, lo, hi in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", operand):
        found |= {(kind, r) for r in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))}
    return found


class Instruction:
    def __init__(self, text, in_asm):
        self.text, self.in_asm = text, in_asm
        self.name, _, rest = text.partition(" ")
        operands = [registers(o) for o in rest.split(",")]
        self.vector = self.name.startswith("v_") and not self.name.startswith("v_cmp")
        self.product = self.name.startswith("v_mfma")
        self.writes = operands[0] if self.vector else set()
        reads = operands[1:]
        if re.match(r"v_(fmac|dot\d+c|mac)", self.name) or "UNUSED_PRESERVE" in text:
            reads = operands
        self.reads = set().union(*reads) if reads else set()
        self.first_source = operands[1] if len(operands) > 1 else set()
        self.states = int(rest) + 1 if self.name == "s_nop" else 1
        self.sub_dword = "dst_sel:" in text and "dst_sel:DWORD" not in text
        self.row = bool(re.search(r"\brow_|\bquad_perm|\bwave_", text))


def functions(assembly):
    """instructions of every function and the places control may come from"""
    for name, body in re.findall(r"^(\w+):\s*; @\w+\n(.*?)^\.Lfunc_end", assembly, re.M | re.S):
        code, labels, in_asm = [], {}, False
        for line in body.split("\n"):
            line = line.strip()
            if line.startswith(";;#ASM"):
                in_asm = line == ";;#ASMSTART"
            elif m := re.match(r"(\.\w+):", line):
                labels[m.group(1)] = len(code)
            elif line and line[0] not in ";.":
                code.append(Instruction(re.sub(r"\s+", " ", line.split(";")[0].strip()), in_asm))
        before = [[i - 1] if i and code[i - 1].name not in ("s_branch", "s_endpgm", "s_setpc_b64") else [] for i in range(len(code) + 1)]
        for i, ins in enumerate(code):
            if ins.name.startswith(("s_branch", "s_cbranch")):
                before[labels[ins.text.split()[1]]].append(i)
        yield name, code, before


def too_close(code, before, at, states, is_bad):
    """does an instruction that is_bad lie fewer than so many wait states before code[at], on any path?"""
    seen, todo = {}, [(p, 0) for p in before[at]]
    while todo:
        i, passed = todo.pop()
        if passed >= states or seen.get(i, states) <= passed:
            continue
        seen[i] = passed
        if is_bad(code[i]):
            return code[i]
        todo += [(p, passed + code[i].states) for p in before[i]]
    return None


def faults(assembly):
    found = []
    for name, code, before in functions(assembly):
        for at, ins in enumerate(code):
            def search(states, is_bad, why):
                other = too_close(code, before, at, states, is_bad)
                if other:
                    found.append(f"{name}: {why}: {other.text}   ...   {ins.text}")
            if ins.in_asm and ins.vector:
                touched = ins.reads | ins.writes
                search(BEHIND_PRODUCT, lambda o: o.product and o.writes & touched, "product and its reader")
                if ins.row:
                    search(BEFORE_ROW, lambda o: o.vector and o.writes & ins.first_source, "row operation")
            if ins.product:
                search(BEFORE_PRODUCT, lambda o: o.in_asm and o.vector and o.writes & ins.reads, "statement and product")
            if ins.vector:
                search(BEHIND_SUBDWORD, lambda o: o.in_asm and o.sub_dword and o.writes & ins.reads, "sub-dword result")
    return found


def wrap(*lines):
    return "f:  ; @f\n" + "\n".join(lines) + "\n\ts_endpgm\n.Lfunc_end0:\n"


def test_the_check_tells_them_apart():
    product, flip = "\tv_mfma_f32_32x32x16_f16 v[0:15], v[16:19], v[20:23], v[0:15]", "v_xor_b32_sdwa v3, v3, v30 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE"
    asm = lambda *l: ("\t;;#ASMSTART", *("\t" + x for x in l), "\t;;#ASMEND")
    assert faults(wrap(product, "\ts_nop 10", *asm(flip)))
    assert not faults(wrap(product, "\ts_nop 11", *asm(flip)))
    assert not faults(wrap(product, *asm(flip.replace("v3", "v33"))))
    assert faults(wrap(*asm(flip), "\ts_nop 0", product))
    assert not faults(wrap(*asm(flip), "\ts_nop 1", product))
    assert faults(wrap(*asm(flip), "\tv_add_f32_e32 v4, v3, v5"))
    assert not faults(wrap(*asm(flip), "\tv_mov_b32_e32 v9, v8", "\tv_add_f32_e32 v4, v3, v5"))
    row = "v_fmac_f32_dpp v40, v41, v42 row_newbcast:1 row_mask:0xf bank_mask:0xf"
    assert faults(wrap("\tv_mov_b32_e32 v41, v1", "\ts_nop 0", *asm(row)))
    assert not faults(wrap("\tv_mov_b32_e32 v41, v1", "\ts_nop 1", *asm(row)))
    # around a loop
    loop = lambda n: wrap("\ts_nop 15", ".LBB0_1:", *asm(flip), "\ts_nop 1", product, f"\ts_nop {n}", "\ts_cbranch_scc1 .LBB0_1")
    assert faults(loop(9)) and not faults(loop(10))


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no compiler")
@pytest.mark.parametrize("source", ["token.hip", "batch.hip", "restore.hip", "panel.hip"])
def test_statements_keep_their_distance_from_products(source, tmp_path):
    from paper_2410_23918_amd import build
    flags = [f for f in build.FLAGS if f != "-shared"]
    out = tmp_path / "kernels.asm"
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", str(CSRC / source), "-o", str(out)], check=True, capture_output=True)
    assembly = out.read_text()
    assert sum(i.in_asm and i.vector for _, code, _ in functions(assembly) for i in code) > 100   # the flips were found
    found = faults(assembly)
    assert not found, "\n".join(found[:10])
