"""Streaming rings read what a neighbour last sent from that neighbour's xhat, with the workgroups
in an order that keeps the three readers of a piece on one L2.  The order is a mapping of its own:
checked here at the counts of tiles where it can go wrong (fewer tiles than XCDs, one more than a
multiple of eight, segments of unequal remainders), whole sends and Top-K, against the oracle."""
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


# elements of the ring's tensors; tiles of 1024 elements (2048 where a Top-K ring's chunks are longer than one)
SIZES = {"one_tile": [5], "seven": [7 * 1024], "eight_and_a_bit": [8 * 1024 + 1], "nine_tensors": [3] * 9,
         "two_segments": [8 * 192 * 1024], "uneven_segments": [8 * 193 * 1024 - 1, 1023, 4097]}


@pytest.mark.parametrize("chunk", [1024, 8192])
@pytest.mark.parametrize("topk", [0, 100_000])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_order_of_the_tiles(evg, oracle_mod, sizes, topk, chunk):
    from helpers import lockstep
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate(SIZES[sizes])]
    w = inputs.Workload("tiles", 3, tensors, 5, sigma0=0.05, fan_in_scaling=1, decay=0.9, topk_ppm=topk, seed=99)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), chunk_elems=chunk, access_mode=evg.ACCESS_STREAM)
    orc = oracle_mod.Oracle.from_workload(w, x0)
    rep = lockstep(ring, orc, w.iters, sample_messages=4)
    assert all(rep["bitwise"].values()), rep
