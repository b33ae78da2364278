"""Assembly statements in the kernels that load: a load that writes registers has to be waited for in the same statement (the
compiler takes an output as written when the statement ends, and may copy, spill or reuse it), and one that writes LDS has to be
a barrier to the compiler's own memory accesses."""
import pathlib
import re

import pytest

SOURCES = sorted((pathlib.Path(__file__).parents[1] / "paper_2410_23918_amd" / "csrc").glob("*.h*"))
LOAD = re.compile(r"\b(?:ds_(?:read|load|bpermute|permute|swizzle)|(?:buffer|global|flat|scratch|s|tbuffer)_(?:load|read))\w*")


def statements(text):
    """(template, the rest) of every asm statement: operands and clobbers are what follows the first colon outside strings"""
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, i, in_string = 1, m.end(), False
        while depth:
            c = text[i]
            if in_string:
                i += c == "\\"
                in_string = c != '"'
            else:
                in_string = c == '"'
                depth += (c == "(") - (c == ")")
            i += 1
        body = text[m.end():i - 1]
        template = re.match(r'\s*(?:"(?:[^"\\]|\\.)*"\s*)+', body).group(0)
        yield "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', template)).replace("\\n", "\n").replace("\\t", " "), body[len(template):]


def faults(text):
    found = []
    for template, rest in statements(text):
        lines = [l.strip() for l in template.split("\n")]
        loads = [i for i, l in enumerate(lines) if LOAD.match(l)]
        to_lds = [i for i in loads if re.search(r"\blds\b", lines[i])]
        if to_lds and '"memory"' not in rest:
            found.append("no memory clobber: " + template)
        to_registers = [i for i in loads if i not in to_lds]
        if to_registers and not any(l.startswith("s_waitcnt") for l in lines[to_registers[-1] + 1:]):
            found.append("no wait after: " + template)
    return found


def test_the_check_tells_them_apart():
    assert faults('asm volatile("ds_read_b128 %0, %1" : "=v"(d) : "v"(a));')
    assert faults('asm volatile("s_waitcnt lgkmcnt(0)\\n\\tds_read_b128 %0, %1" : "=v"(d) : "v"(a));')
    assert not faults('asm volatile("ds_read_b128 %0, %1\\n\\ts_waitcnt lgkmcnt(0)" : "=v"(d) : "v"(a));')
    assert faults('asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(o), "s"(r));')
    assert not faults('asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(o), "s"(r) : "memory");')
    assert not faults('asm("v_mov_b32 %0, %1" : "=v"(d) : "v"(a));')


@pytest.mark.parametrize("path", SOURCES, ids=lambda p: p.name)
def test_loads_in_assembly_are_waited_for_in_place(path):
    assert not faults(path.read_text())
