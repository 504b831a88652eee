"""The walking pass of Top-K rings deals its windows to the XCDs in contiguous eighths, by a mapping of its own from a workgroup's
number to its window: checked at the counts of windows where it can go wrong (fewer than XCDs, a multiple of eight, one
more, one less, last eighths that are short or empty), whole sends, whose windows are taken in turn, beside it,
against the oracle."""
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


# elements of the ring's tensors.  Windows of 1024 elements with chunks of 1024, of 2048 with chunks of 2048 (and four to every chunk of
# 8192): 1, 7, 8, 9, 15, 17 and 65 of them, tensors of one element among them, and many
SIZES = {"one": [5], "seven": [7 * 1024], "eight": [8 * 1024], "eight_and_a_bit": [8 * 1024 + 1], "nine_tensors": [3] * 9,
         "fifteen": [14 * 1024, 1], "seventeen": [15 * 2048, 1, 1], "sixty_five": [3] * 64 + [2047], "many": [193 * 1024 - 1, 1023, 4097]}


@pytest.mark.parametrize("chunk", [1024, 2048, 8192])
@pytest.mark.parametrize("topk", [0, 100_000])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_order_of_the_windows(evg, oracle_mod, sizes, topk, chunk):
    from helpers import lockstep
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate(SIZES[sizes])]
    w = inputs.Workload("windows", 3, tensors, 5, sigma0=0.05, fan_in_scaling=1, decay=0.9, topk_ppm=topk, seed=99)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), chunk_elems=chunk, access_mode=evg.ACCESS_STREAM)
    orc = oracle_mod.Oracle.from_workload(w, x0)
    rep = lockstep(ring, orc, w.iters, sample_messages=4)
    assert all(rep["bitwise"].values()), rep
