"""The decomposition's row operations in assembly (the substitution of k_dc_orth), searched like the other kernels' statements."""
import shutil
import subprocess

import pytest

from test_asm_distances import CSRC, HIPCC, faults, functions


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no compiler")
def test_row_operations_keep_their_distance(tmp_path):
    from paper_2410_23918_amd import build
    out = tmp_path / "kernels.asm"
    subprocess.run([HIPCC, *[f for f in build.FLAGS if f != "-shared"], "--cuda-device-only", "-S", str(CSRC / "decompose.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    assembly = out.read_text()
    assert sum(i.in_asm and i.row for _, code, _ in functions(assembly) for i in code) == 31 * 32 // 2
    found = faults(assembly)
    assert not found, "\n".join(found[:10])
