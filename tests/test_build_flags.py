"""Compiler options that the kernels' values depend on (build_lib.FLAGS)."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09772_amd import build_lib

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_spills_are_not_split_over_registers(tmp_path):
    """No value of a kernel that spills is kept half in a spare register and
    half in scratch: the compiler loses the register half of such a value when
    it comes back into an accumulation register pair."""
    src = tmp_path / "k.hip"
    src.write_text(f'#include "{build_lib.CSRC}/jk_registry.h"\n#include "{build_lib.CSRC}/jk_device.h"\n'
                   "namespace jk {\ntemplate __global__ void jk_k1_row<3, 1, 2, 0, float, 256>(const JkArgs, const ClsArgs *, "
                   "const ClsGroup, const BatchDesc *, int);\n}\n")
    asm = tmp_path / "k.s"
    subprocess.run([HIPCC, *build_lib.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True)
    text = asm.read_text()
    assert "Folded Spill" in text and "Folded Reload" in text
    assert "Reload Reuse" not in text
