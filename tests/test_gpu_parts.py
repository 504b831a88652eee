"""Cached rings that send whole tensors are updated in parts of the ring, one workgroup to a window and a part, or (most of those here
of at most 16 workers) one to a window of the whole ring; test_gpu_passes.py says which and has the rings of the other pass.  Checked
against the oracle at closed rings of 3 to 8 workers, last parts of one worker or a few, with and without a tensor whose tests need a launch of their own, and replayed from a graph, in
whose launches every workgroup keeps count of the iterations by itself."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

ARENAS = ("x", "xhat", "vel", "mbox_l", "mbox_r")
LONG = 128 * 1024 + 1


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _workload(P, sizes, iters, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate(sizes)]
    return inputs.Workload("parts", P, tensors, iters, sigma0=0.05, decay=0.9, seed=P, **kw)


# 17 workers, and 13 and 16 that draw: parts, of 4 and 8; the others whole rings
@pytest.mark.parametrize("P,sizes", [(3, [1300, 7, 2048]), (4, [1023, 1, 5]), (5, [1025, 3]), (9, [4097, 2]),
                                     (3, [1021] * 310), (4, [3] * 300), (9, [1027] * 90), (17, [5] * 100),
                                     (8, [2] * 520), (9, [3] * 430), (11, [1] * 400), (16, [1023] * 240),
                                     (3, [LONG, 9]), (6, [LONG + 2, 3]), (13, [LONG, 70])])
@pytest.mark.parametrize("kw", [dict(spike_prob=0.3, spike_gain=4.0), dict(momentum=0.0, dist=1), dict(trigger_kind=1)],
                         ids=["normal", "student_plain", "norms"])
def test_parts(evg, oracle_mod, P, sizes, kw):
    from helpers import lockstep
    kw = dict(kw)
    both = dict(trigger_kind=kw.pop("trigger_kind")) if "trigger_kind" in kw else {}
    w = _workload(P, sizes, 6, **kw)
    x0 = inputs.replicate(w.x0(), P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), **both)
    orc = oracle_mod.Oracle.from_workload(w, x0, **both)
    rep = lockstep(ring, orc, w.iters, sample_messages=0, norm_rtol=None if both else 2e-7, norm_abs_of_x=2.5e-7 if both else None)
    assert rep["rel"]["x"] <= 1e-5 and (both or all(rep["bitwise"].values())), rep


@pytest.mark.parametrize("P,sizes", [(4, [1300, 7]), (9, [1027] * 90), (9, [3] * 430), (5, [LONG, 3])])
@pytest.mark.parametrize("trigger_kind", [0, 1])
def test_replays_of_a_graph_that_outlive_an_import(evg, P, sizes, trigger_kind):
    import torch
    w = _workload(P, sizes, 0, spike_prob=0.3, spike_gain=4.0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = evg.Ring.from_workload(w, mailbox_fill=0.0, stream=stream, trigger_kind=trigger_kind)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, trigger_kind=trigger_kind)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step_next()
    for k in range(3):                     # (the capture itself runs nothing)
        g.replay()
        b.step(k)
    torch.cuda.synchronize()
    ck = b.export_state()                  # after an odd number of steps
    for k in range(3, 7):
        g.replay()
        b.step(k)
        torch.cuda.synchronize()
        assert np.array_equal(a.decisions()["fired"], b.decisions()["fired"]), k
    for name in ARENAS:
        assert np.array_equal(a.state(name), b.state(name)), name
    a.import_state(ck)
    b.import_state(ck)
    for k in range(3, 6):
        g.replay()
        b.step(k)
    a.step(6)
    b.step(6)
    g.replay()
    b.step(7)
    torch.cuda.synchronize()
    da, db = a.decisions(), b.decisions()
    assert all(np.array_equal(da[key], db[key]) for key in da)
    assert a.stats()["iters"] == b.stats()["iters"] == 8
    for name in ARENAS:
        assert np.array_equal(a.state(name), b.state(name)), name
