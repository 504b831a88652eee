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


def test_whole_rings_count_behind_a_barrier(tmp_path):
    """The counts of key codes are cleared by all wavefronts of a workgroup together: none adds to them before a barrier behind that."""
    counting = 0
    for m in re.finditer(r"^(_ZN3evg13k_update_ring\w+):(.*?)^\.Lfunc_end", _assembly(tmp_path, "kernels_ring.hip"), re.M | re.S):
        order = re.findall(r"^\s+(ds_write_b32|ds_add_u32|s_barrier)\b", m.group(2), re.M)
        if "ds_add_u32" in order:
            counting += 1
            assert order[0] == "ds_write_b32" and "s_barrier" in order[:order.index("ds_add_u32")], (m.group(1), order[:4])
    assert counting == 12          # three gradients, two norms, windows of two sizes
