"""k_topk_choose on the CPU (emulated_wavefronts.h): between two barriers a workgroup's wavefronts may run in any order, so the selection
has to be the same whichever goes first.  Ties that do not all win, near ones, lists that overflow, several rounds over a tensor's groups, no key
codes, and a tensor of one wavefront."""
import os
import subprocess

import pytest

from paper_2103_07454_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.fixture(scope="module")
def selection(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("compiles device code as C++")
    d = tmp_path_factory.mktemp("choose")
    os.mkdir(d / "hip")
    (d / "hip" / "hip_runtime.h").write_text('#pragma once\n#include "emulated_wavefronts.h"\n')
    with open(os.path.join(build.CSRC, "kernels_choose.hip")) as f:
        text = f.read()
    lds = "extern __shared__ uint32_t groups[];"
    assert text.count(lds) == 1 and text.count("hipError_t launch_topk_choose") == 1
    text = text[:text.index("hipError_t launch_topk_choose")] + "}  // namespace evg\n"
    (d / "kernels_choose.hip").write_text(text.replace(lds, "uint32_t* const groups = emu::dynamic_lds.data();"))
    exe = d / "choose"
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", f"-I{d}", f"-I{HERE}", f"-I{build.CSRC}",
                    "-o", str(exe), os.path.join(HERE, "choose_workgroups.cpp")], check=True)
    return exe


# (elements, K, keys equal to the K-th largest, others just below, key codes) and whether the selection goes by the codes
@pytest.mark.parametrize("n,K,ties,near,codes,staged", [
    (200, 20, 7, 2, 1, 1), (257, 26, 1, 0, 1, 1), (5000, 500, 40, 0, 1, 1), (9000, 900, 100, 9, 1, 1), (300_000, 30_000, 1, 3, 1, 1),
    (300_000, 30_000, 30, 90, 1, 1), (300_000, 30_000, 900, 5, 1, 1), (600_000, 60_000, 3000, 9, 1, 1), (300_000, 30_000, 5000, 0, 1, 0),
    (300_000, 3000, 300, 0, 0, 0)])
def test_any_wavefront_may_go_first(selection, n, K, ties, near, codes, staged):
    out = subprocess.run([str(selection), *map(str, (n, K, ties, near, codes))], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == f"ok equal {ties} staged {staged}\n", out.stdout + out.stderr
