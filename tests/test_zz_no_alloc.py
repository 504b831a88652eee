"""evg_init_static: the variant of evg_init for callers that must not allocate device memory.
Its contexts must behave exactly like evg_init's: two rings in a row share the GPU's static
scratch block, the second smaller than the first (so it finds the first one's leftovers), and
each is compared bit for bit, iteration by iteration, with a ring created by evg_init."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

ARENAS = ("x", "xhat", "vel", "mbox_l", "mbox_r")


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    # the HIP runtime places the library's code object and its static scratch block on the GPU
    # when they are first used (the set-up of the first evg_init_static on a device looks the
    # block's address up); do that once before free device memory is compared
    w = workload(3, [64])
    r = m.Ring.from_workload(w, inputs.replicate(w.x0(), w.P), static_tables=True)
    r.step(0)
    r.synchronize()
    r.close()
    return m


def workload(P, sizes, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 8 + i, "weight") for i, n in enumerate(sizes)]
    base = dict(sigma0=0.05, fan_in_scaling=1, decay=0.98, seed=77)
    base.update(kw)
    return inputs.Workload("static", P, tensors, 14, **base)


def run_pair(evg, w, iters, same_tables=True, **over):
    import torch
    x0 = inputs.replicate(w.x0(), w.P)
    a = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), static_tables=True, **over)
    # free device memory did not move across evg_init_static: the library took nothing
    assert a.library_bytes == 0, a.library_bytes
    b = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), **over)
    for k in range(iters):
        a.step(k)
        b.step(k)
        da, db = a.decisions(), b.decisions()
        for name in ("fired", "near_tie", "norm", "delta_before"):
            assert np.array_equal(da[name], db[name], equal_nan=True), (k, name)
        if w.topk_ppm:
            ha, hb = a.message_hashes(), b.message_hashes()
            assert np.array_equal(ha[0], hb[0]) and np.array_equal(ha[1], hb[1]), k
    sa, sb = a.stats(arrays=True), b.stats(arrays=True)
    for key in sa:
        if same_tables or key not in ("library_bytes", "chunks_not_staged"):
            assert np.array_equal(sa[key], sb[key]), key
    assert sa["events_total"] > w.P * w.L
    for name in ARENAS:
        ta, tb = getattr(a, name), getattr(b, name)
        idx = torch.from_numpy(a.layout.index).to(ta.device)
        assert torch.equal(ta.index_select(1, idx).view(torch.int32), tb.index_select(1, idx).view(torch.int32)), name
    assert np.array_equal(a.average(), b.average())
    b.close()
    return a


def test_static_tables_match_allocated_tables_twice_in_a_row(evg):
    # first ring: Top-K messages, ragged tensors over several chunks
    w1 = workload(6, [20000, 1, 4097, 9000, 7, 1024], topk_ppm=100_000)
    a1 = run_pair(evg, w1, 14)
    # a second static context on the same GPU is refused while the first one lives
    w2 = workload(4, [5000, 3, 1300], spike_prob=0.2, spike_gain=5.0)
    x2 = inputs.replicate(w2.x0(), w2.P)
    with pytest.raises(evg.EvgError) as ei:
        evg.Ring.from_workload(w2, x2, static_tables=True)
    assert ei.value.status == 5
    a1.close()
    # second ring, smaller, other options: the block still holds the first ring's tables
    a2 = run_pair(evg, w2, 14)
    a2.close()
    # third: Top-K again, smaller than the first, with the history-averaged threshold
    w3 = workload(3, [3000, 513], topk_ppm=50_000)
    a3 = run_pair(evg, w3, 14, hist_len=3)
    a3.close()


def test_configuration_beyond_the_block_is_rejected(evg):
    w = workload(8, [3_000_000], topk_ppm=100_000)     # staging alone would take 3 x 96 MB
    x0 = inputs.replicate(w.x0(), w.P)
    with pytest.raises(evg.EvgError) as ei:
        evg.Ring.from_workload(w, x0, static_tables=True)
    assert ei.value.status == 1 and "static scratch block" in str(ei.value)
    # ... and the block is free again afterwards
    w2 = workload(3, [100, 5])
    r = evg.Ring.from_workload(w2, inputs.replicate(w2.x0(), w2.P), static_tables=True)
    r.step(0)
    r.synchronize()
    r.close()


# What is admitted does not change with the tables' present sizes: one long tensor, many tiny ones, whole sends of many
# tensors, each at the last size that has always been admitted and at the first that never was.  (The chunks may be shorter
# than evg_init's; a state blob goes either way all the same.)
@pytest.mark.parametrize("P,most,more,kw,over", [
    (8, [2_178_496], [2_178_560], dict(topk_ppm=100_000), dict(chunk_elems=8192)),
    (3, [4] * 2630, [4] * 2631, dict(topk_ppm=100_000), dict(chunk_elems=8192)),
    (16, [4] * 62_112, [4] * 62_113, dict(), dict(chunk_elems=1024, access_mode=1)),
    # (a cached ring, and one with so many tensors that what its update in parts takes has no room)
    (16, [15] * 18_332, [15] * 18_333, dict(), dict(access_mode=2)),
    (16, [15] * 18_332, [15] * 20_166, dict(), dict(access_mode=2))], ids=["long", "tiny", "whole", "cached", "cached_no_parts"])
def test_the_largest_configurations_admitted(evg, P, most, more, kw, over):
    with pytest.raises(evg.EvgError) as ei:
        evg.Ring.from_workload(workload(P, more, **kw), static_tables=True, **over)
    assert ei.value.status == 1 and "static scratch block" in str(ei.value)
    w = workload(P, most, **kw)
    a = run_pair(evg, w, 5, same_tables=False, **over)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, **over)
    b.import_state(a.export_state())
    for k in range(5, 8):
        a.step(k)
        b.step(k)
    a.import_state(b.export_state())
    for k in range(8, 10):
        a.step(k)
        b.step(k)
    assert np.array_equal(a.decisions()["fired"], b.decisions()["fired"])
    for name in ARENAS:
        assert np.array_equal(a.state(name), b.state(name)), name
    a.close()
    b.close()


def test_where_a_sum_a_group_has_no_room_parts_of_the_ring_do(evg):
    w = workload(12, [4] * 36_000)
    a = run_pair(evg, w, 4, same_tables=False)
    b = evg.Ring.from_workload(w)
    assert a.update_pass() == ("k_update_part", 8, 1024) and b.update_pass()[0] == "k_update_ring"
    a.close()
    b.close()
