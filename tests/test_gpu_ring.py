"""Cached rings of at most 16 workers, and streaming ones with whole sends, are updated by one workgroup for each window of the whole
ring; windows are of 256, 512 or 1024 elements, and a thread has one float4 or a few.  Checked against the oracle at the edges of groups, windows and chunks,
by sizes that lead to each shape of a workgroup (evg_api.hip: ring_shape, stream_shape)."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

EDGES = [255, 256, 257, 511, 513, 1023, 1025, 2047, 2049, 1, 4]


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _workload(P, sizes, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i % 40, "weight") for i, n in enumerate(sizes)]
    return inputs.Workload("ring", P, tensors, 7, sigma0=0.05, decay=0.9, seed=P, **kw)


def _check(evg, oracle_mod, w, both=None, given=False, **gpu):
    import torch
    from helpers import lockstep
    both = both or {}
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), grad_mode=int(given), **both, **gpu)
    orc = oracle_mod.Oracle.from_workload(w, x0, grad_mode=int(given), **both)
    host = dev = None
    if given:
        def host(k):
            return inputs.random_grads(w.P, w.N, 40 + k, 0.02)

        def dev(k):
            return torch.from_numpy(ring.layout.pad(host(k))).cuda()
    norms = both.get("trigger_kind", 0)
    rep = lockstep(ring, orc, w.iters, grads=host, gpu_grads=dev, sample_messages=3,
                   norm_rtol=None if norms else 2e-7, norm_abs_of_x=2.5e-7 if norms else None)
    assert rep["rel"]["x"] <= 1e-5 and (norms or all(rep["bitwise"].values())), rep


# one float4 a thread (short windows; with a tensor of more than 65 536 elements longer ones), two, whole sweeps
WHOLE = [(3, EDGES), (13, EDGES * 6), (5, EDGES + [65537, 131072]), (8, EDGES * 10), (12, EDGES * 8), (16, [1023] * 200 + EDGES * 4),
         (3, EDGES * 25), (4, EDGES * 25), (6, EDGES * 10 + [131073])]


@pytest.mark.parametrize("P,sizes", WHOLE, ids=[f"{P}x{len(s)}" for P, s in WHOLE])
@pytest.mark.parametrize("kw", [dict(spike_prob=0.3, spike_gain=4.0), dict(momentum=0.0, dist=1), dict(trigger_kind=1), dict(given=True)],
                         ids=["normal", "student_plain", "norms", "given"])
def test_whole_sends(evg, oracle_mod, P, sizes, kw):
    kw = dict(kw)
    both = {k: kw.pop(k) for k in ("trigger_kind",) if k in kw}
    given = kw.pop("given", False)
    _check(evg, oracle_mod, _workload(P, sizes, **kw), both, given)


TOPK = [(5, EDGES * 24), (12, EDGES * 10 + [5000]), (16, [700] * 200 + EDGES * 4), (13, [257] * 300 + EDGES)]


@pytest.mark.parametrize("P,sizes", TOPK, ids=[f"{P}x{len(s)}" for P, s in TOPK])
@pytest.mark.parametrize("kw", [dict(topk_ppm=100_000), dict(topk_ppm=3_000, momentum=0.0, dist=1), dict(topk_ppm=400_000, trigger_kind=1),
                                dict(topk_ppm=100_000, given=True)], ids=["normal", "student_plain", "norms", "given"])
def test_messages(evg, oracle_mod, P, sizes, kw):
    kw = dict(kw)
    both = {k: kw.pop(k) for k in ("trigger_kind",) if k in kw}
    given = kw.pop("given", False)
    _check(evg, oracle_mod, _workload(P, sizes, **kw), both, given)


# a blob holds a sum for every 1024 elements, however many windows a ring has there
@pytest.mark.parametrize("sizes", [EDGES, EDGES * 12, EDGES * 25], ids=len)
@pytest.mark.parametrize("kw", [dict(), dict(trigger_kind=1), dict(topk_ppm=100_000)], ids=["whole", "norms", "topk"])
def test_checkpoints_with_short_windows(evg, sizes, kw):
    kw = dict(kw)
    both = {k: kw.pop(k) for k in ("trigger_kind",) if k in kw}
    w = _workload(4, sizes, **kw)
    rings = [evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=m, **both) for m in (evg.ACCESS_CACHED, evg.ACCESS_STREAM)]
    for k in range(5):
        for r in rings:
            r.step(k)
    blobs = [r.export_state() for r in rings]
    others = [evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=m, **both) for m in (evg.ACCESS_STREAM, evg.ACCESS_CACHED)]
    for r, b in zip(others, blobs):
        r.import_state(b)
    for k in range(5, 9):
        for r in rings + others:
            r.step(k)
        for r in rings[1:] + others:
            assert np.array_equal(r.decisions()["fired"], rings[0].decisions()["fired"]), k
    for r in rings[1:] + others:
        for name in ("x", "xhat", "vel", "mbox_l", "mbox_r"):
            assert np.array_equal(r.state(name), rings[0].state(name)), name


# streaming rings: windows that begin on cache lines, workgroups of every shape (8, 16, 32 workers and more), tensors shorter than their lead
STREAMED = [(3, EDGES), (8, EDGES * 3 + [8191, 8193, 20_001]), (9, EDGES * 2), (16, [5, 31, 33] + EDGES), (17, EDGES), (32, [1000, 3, 8192]), (33, [1021, 7]),
            (64, [257, 2, 513])]


@pytest.mark.parametrize("P,sizes", STREAMED, ids=[f"{P}x{len(s)}" for P, s in STREAMED])
@pytest.mark.parametrize("kw", [dict(spike_prob=0.3, spike_gain=4.0), dict(momentum=0.0, dist=1), dict(trigger_kind=1), dict(given=True)],
                         ids=["normal", "student_plain", "norms", "given"])
def test_streamed_whole_sends(evg, oracle_mod, P, sizes, kw):
    kw = dict(kw)
    both = {k: kw.pop(k) for k in ("trigger_kind",) if k in kw}
    given = kw.pop("given", False)
    _check(evg, oracle_mod, _workload(P, sizes, **kw), both, given, access_mode=evg.ACCESS_STREAM)


@pytest.mark.parametrize("P", [5, 16, 40])
def test_replays_of_streamed_steps(evg, P):
    import torch
    w = _workload(P, EDGES, spike_prob=0.3, spike_gain=4.0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = evg.Ring.from_workload(w, mailbox_fill=0.0, stream=stream, access_mode=evg.ACCESS_STREAM)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=evg.ACCESS_STREAM)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step_next()
    for k in range(6):
        g.replay()
        b.step(k)
        torch.cuda.synchronize()
        assert np.array_equal(a.decisions()["fired"], b.decisions()["fired"]), k
    for name in ("x", "xhat", "vel", "mbox_l", "mbox_r"):
        assert np.array_equal(a.state(name), b.state(name)), name


# the sums that the next test reads come back as they were, and so does all that follows from them
@pytest.mark.parametrize("P,sizes,stream", [(3, EDGES * 6, False), (5, EDGES * 4 + [65537], False), (8, EDGES * 10, False), (3, EDGES * 25, False),
                                            (8, EDGES * 3 + [20_001], True), (16, EDGES * 3, True), (40, EDGES, True)])
@pytest.mark.parametrize("kw", [dict(), dict(trigger_kind=1), dict(topk_ppm=100_000), dict(topk_ppm=100_000, trigger_kind=1)],
                         ids=["whole", "norms", "topk", "norms_topk"])
def test_a_resumed_ring_goes_on_bit_for_bit(evg, P, sizes, stream, kw):
    kw = dict(kw)
    over = {k: kw.pop(k) for k in ("trigger_kind",) if k in kw}
    w = _workload(P, sizes, **kw)
    a, b = (evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=evg.ACCESS_STREAM if stream else evg.ACCESS_CACHED, **over) for _ in range(2))
    for k in range(4):
        a.step(k)
    b.import_state(a.export_state())
    for k in range(4, 9):
        a.step(k)
        b.step(k)
        da, db = a.decisions(), b.decisions()
        for name in ("fired", "norm", "delta_before"):
            assert np.array_equal(da[name].view(np.uint8), db[name].view(np.uint8)), (k, name)
        ba, bb = a.export_state(), b.export_state()
        end = len(ba["blob"]) - (P * len(sizes) * 2048 * 4 if "topk_ppm" in kw else 0)      # (behind it the counts of keys, whose cut into bins may differ)
        assert np.array_equal(ba["blob"][:end], bb["blob"][:end]), k
    for name in ("x", "xhat", "vel", "mbox_l", "mbox_r"):
        assert np.array_equal(a.state(name), b.state(name)), name


# the shapes that ring_shape and stream_shape choose for the rings above, and the other passes at their edges
@pytest.mark.parametrize("P,sizes,kw,stream,given,want", [
    (3, EDGES, {}, False, False, ("k_update_ring", 3, 256)), (5, EDGES + [65537], {}, False, False, ("k_update_ring", 5, 512)),
    (3, EDGES * 25, {}, False, False, ("k_update_ring", 3, 1024)), (12, EDGES * 10 + [5000], dict(topk_ppm=100_000), False, False, ("k_update_ring", 12, 512)),
    (16, [700] * 200 + EDGES * 4, dict(topk_ppm=100_000), False, True, ("k_update_ring", 16, 256)),
    (17, EDGES, {}, False, False, ("k_update_part", 2, 1024)), (8, EDGES, {}, True, False, ("k_update_ring", 8, 512)),
    (9, EDGES, {}, True, False, ("k_update_ring", 9, 256)), (65, EDGES, {}, True, False, ("k_update_walk", 1, 0)),
    (5, EDGES, dict(topk_ppm=100_000), True, False, ("k_update_walk", 5, 0)),
    (7, EDGES + [65537], {}, False, False, ("k_update_ring", 7, 256)), (4, [200] * 450, {}, False, True, ("k_update_ring", 4, 256)),
    (8, [1000] * 505, {}, False, False, ("k_update_part", 8, 1024)), (8, [1000] * 505, dict(dist=1), False, False, ("k_update_ring", 8, 512)),
    (8, [1100] * 260, {}, False, False, ("k_update_ring", 8, 512)), (8, [1000] * 370 + [140_000], {}, False, False, ("k_update_ring", 8, 512)),
    (10, [1000] * 260, {}, False, False, ("k_update_part", 4, 1024)), (10, [1000] * 260, {}, False, True, ("k_update_ring", 10, 512)),
    (12, [1000] * 290, {}, False, False, ("k_update_ring", 12, 512)), (13, [1000] * 320, {}, False, False, ("k_update_part", 8, 1024)),
    (13, [1000] * 320, dict(dist=1), False, False, ("k_update_ring", 13, 512)),
    (13, [1000] * 320, dict(dist=1, spike_prob=0.1), False, False, ("k_update_part", 8, 1024)), (13, [300] * 320, {}, False, False, ("k_update_ring", 13, 512)), (13, [320_000, 9], {}, False, False, ("k_update_ring", 13, 512)),
    (13, [360_000, 9], dict(dist=1), False, False, ("k_update_part", 4, 1024)),
    (13, [64_000, 10], {}, False, True, ("k_update_ring", 13, 256)), (13, [2000] * 66, {}, False, True, ("k_update_part", 4, 1024)),
    (13, [2000] * 150, {}, False, True, ("k_update_ring", 13, 512)), (10, [1000] * 280, dict(topk_ppm=100_000), False, False, ("k_update_part", 4, 1024)),
    (10, [300] * 280, dict(topk_ppm=100_000), False, False, ("k_update_ring", 10, 512)), (10, [1000] * 280, dict(topk_ppm=100_000), False, True, ("k_update_ring", 10, 512))], ids=lambda v: f"{len(v)} tensors" if isinstance(v, list) else str(v))
def test_the_pass_chosen(evg, P, sizes, kw, stream, given, want):
    ring = evg.Ring.from_workload(_workload(P, sizes, **kw), grad_mode=int(given), access_mode=evg.ACCESS_STREAM if stream else evg.ACCESS_AUTO)
    assert ring.update_pass() == want


# streaming whole sends: where the slices of more than eight workers lie multiples of 8 KB apart, or up to 256 bytes more or less, and where more than 32 workers have
# mostly one long tensor, rings are walked; all others of up to 64 workers are not
@pytest.mark.parametrize("P,sizes,walked", [(9, [16_384 + d], abs(d) < 128) for d in (-128, -64, 0, 64, 128)] + [
    (8, [16_384], False), (64, [16_384 - 64], True), (64, [16_384 - 128], False), (33, [262_144, 1000], False), (33, [262_148, 1000], True),
    (32, [262_148, 1000], False), (33, [262_148, 262_148, 1000], False)], ids=lambda v: str(v).replace(" ", ""))
def test_the_streamed_rings_that_are_walked(evg, P, sizes, walked):
    ring = evg.Ring.from_workload(_workload(P, sizes), access_mode=evg.ACCESS_STREAM)
    assert (ring.update_pass()[0] == "k_update_walk") == walked
