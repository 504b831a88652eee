"""What can be told from the device code that hipcc makes, without a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2103_07454_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="reads what hipcc compiles")


def _assembly(tmp_path, source):
    out = tmp_path / "device.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    return out.read_text()


def test_short_tensors_are_tested_by_as_many_wavefronts_as_a_simd_holds(tmp_path):
    registers = {m.group(1): int(m.group(2)) for m in re.finditer(r"\.amdhsa_kernel (_ZN3evg9k_trigger\w+).*?\.amdhsa_next_free_vgpr (\d+)",
                                                                  _assembly(tmp_path, "kernels_trigger.hip"), re.S)}
    assert len(registers) == 2 and sorted(registers.values())[0] <= 64, registers
