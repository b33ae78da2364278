"""Assembly statements of decompose.hip (the row operations of k_dc_orth's substitution) and rows.hip, searched like the other kernels'."""
import shutil
import subprocess

import pytest

from test_asm_distances import CSRC, HIPCC, faults, functions


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no compiler")
@pytest.mark.parametrize("source", ["decompose.hip", "rows.hip"])
def test_statements_keep_their_distance(source, tmp_path):
    from paper_2410_23918_amd import build
    out = tmp_path / "kernels.asm"
    subprocess.run([HIPCC, *[f for f in build.FLAGS if f != "-shared"], "--cuda-device-only", "-S", str(CSRC / source), "-o", str(out)],
                   check=True, capture_output=True)
    assembly = out.read_text()
    statements = [i for _, code, _ in functions(assembly) for i in code if i.in_asm and i.vector]
    assert sum(i.row for i in statements) == 31 * 32 // 2 if source == "decompose.hip" else len(statements) > 100   # they were found
    found = faults(assembly)
    assert not found, "\n".join(found[:10])
