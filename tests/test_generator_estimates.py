"""The gradient generator's quotients and roots: a hardware estimate and one correction.  On the CPU, over all 2^23 uniforms:
with a correctly rounded estimate the correction gives what the IEEE operators give, and with one that is a unit in the last
place off it does so for all but the few uniforms of WORDS.  Those are drawn on the GPU, at counters found by search,
and compared with the oracle, which uses the operators: together every radius the generator can draw."""
import os
import subprocess

import numpy as np
import pytest

from paper_2103_07454_amd import inputs

SEED = 0x2103
# distribution (0 normal, 1 Student-t), uniform, and a place in the stream where it is the radius: iteration, worker, block, word
WORDS = [
    (0, 4194303, 571, 1, 782, 2), (0, 1554824, 645, 0, 588, 2), (0, 5619991, 698, 2, 903, 2), (0, 6085852, 866, 1, 254, 2),
    (0, 4047135, 1501, 2, 130, 0), (0, 5264077, 2481, 0, 679, 2), (0, 1550773, 4028, 1, 395, 2),
    (1, 4194303, 571, 1, 782, 2), (1, 1554824, 645, 0, 588, 2), (1, 6085852, 866, 1, 254, 2), (1, 5881792, 867, 2, 382, 2),
    (1, 2820504, 960, 2, 665, 2), (1, 215022, 1363, 0, 250, 2), (1, 1215070, 1402, 2, 121, 2), (1, 4047135, 1501, 2, 130, 0),
    (1, 1550773, 4028, 1, 395, 2)]


def test_uniforms_at_which_an_estimate_counts(tmp_path):
    exe = tmp_path / "estimates"
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "generator_estimates.cpp")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-o", str(exe), src], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    assert not [line for line in out if line.startswith("general")]
    assert {tuple(map(int, line.split())) for line in out if line} == {(d, n) for d, n, *_ in WORDS}


def test_the_uniforms_lie_where_stated(oracle_mod):
    for _, n, k, r, block, word in WORDS:
        assert oracle_mod.philox4x32_10([block, 0, k, r], [SEED, 0])[word] >> 9 == n


@pytest.mark.gpu
@pytest.mark.parametrize("dist", [0, 1])
def test_they_are_drawn_as_the_oracle_draws_them(oracle_mod, dist):
    """lr = 1, no momentum, x0 = 0, no communication: x = -g after one step."""
    from paper_2103_07454_amd import evg
    w = inputs.Workload("words", 3, [inputs.TensorSpec("a", (4096,), 1, "weight")], 1, lr=1.0, momentum=0.0,
                        thr_mode=inputs.THR_FIXED, thr_fixed=float("inf"), force_first=0, dist=dist, sigma0=1.0, fan_in_scaling=0,
                        decay=1.0, seed=SEED)
    x0 = np.zeros((w.P, w.N), np.float32)
    for d, n, k, r, block, word in WORDS:
        if d != dist:
            continue
        ring, orc = evg.Ring.from_workload(w, x0), oracle_mod.Oracle.from_workload(w, x0)
        ring.step(k)
        orc.step(k)
        got, want = ring.state("x"), orc.state("x")
        j = 4 * block + word if dist == 0 else 4 * (block // 2) + 2 * (block % 2) + word // 2
        assert got[r, j] != 0 and got[r, j].view(np.uint32) == want[r, j].view(np.uint32), (n, got[r, j], want[r, j])
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
        ring.close()
