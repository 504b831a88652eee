"""Every update pass, at rings that the present rules send to it (evg_api.hip: ring_shape, stream_shape): which pass it is and what a workgroup has is
asserted, so that a later rule cannot lead a test past what it is for.  Against the oracle, with drawn and given gradients and both triggers: parts of the ring of
1, 2, 4 and 8 workers, last parts of one and some, closed rings; windows of 256, 512 and 1024 elements of the whole ring; whole sends of walked rings, in parts and in
one.  And replayed from a graph, also after an import."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

ARENAS = ("x", "xhat", "vel", "mbox_l", "mbox_r")
EDGES = [255, 256, 257, 511, 513, 1023, 1025, 2047, 2049, 1, 4]
LONG = 128 * 1024 + 1
OPTIONS = dict(normal=dict(spike_prob=0.3, spike_gain=4.0), student_plain=dict(momentum=0.0, dist=1), norms=dict(trigger_kind=1), given=dict(given=True))


def _on_8k(sizes):
    """With a last tensor that makes workers lie a multiple of 8 KB apart."""
    n = sum(-(-s // 4) * 4 for s in sizes)
    return sizes + [2048 - n % 2048]


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _workload(P, sizes, iters, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i % 40, "weight") for i, n in enumerate(sizes)]
    return inputs.Workload("passes", P, tensors, iters, sigma0=0.05, decay=0.9, seed=P, **kw)


def _check(evg, oracle_mod, P, sizes, want, options, *, iters=5, **kw):
    import torch
    from helpers import lockstep
    options = dict(options)
    both = {k: options.pop(k) for k in ("trigger_kind",) if k in options}
    given = options.pop("given", False)
    w = _workload(P, sizes, iters, **options, **{k: kw.pop(k) for k in ("topk_ppm",) if k in kw})
    x0 = inputs.replicate(w.x0(), P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), grad_mode=int(given), **both, **kw)
    assert ring.update_pass() == want
    orc = oracle_mod.Oracle.from_workload(w, x0, grad_mode=int(given), **both)
    grads = {k: inputs.random_grads(P, w.N, 40 + k, 0.02) for k in range(iters if given else 0)}
    on_gpu = {k: torch.from_numpy(ring.layout.pad(g)).cuda() for k, g in grads.items()}
    rep = lockstep(ring, orc, iters, grads=grads.get if given else None, gpu_grads=on_gpu.get if given else None, sample_messages=4,
                   norm_rtol=None if both else 2e-7, norm_abs_of_x=2.5e-7 if both else None)
    assert rep["rel"]["x"] <= 1e-5 and (both or all(rep["bitwise"].values())), rep


# few windows: parts of 2; some 100: of 4; some 200: of 8; a tensor whose tests need a launch of their own: 4 at most
PARTS = [(17, [1300, 7, 2048], 2), (17, [5] * 20, 2), (19, [5] * 100, 4), (24, [1027] * 60, 4), (33, [3] * 110, 8), (18, [1027] * 100, 8), (19, [LONG, 3], 4),
         (4, [3] * 720, 4), (3, [3] * 1150, 3), (14, [1027, 3] * 30, 4)]


@pytest.mark.parametrize("P,sizes,part", PARTS, ids=[f"{p[0]}x{len(p[1])}" for p in PARTS])
@pytest.mark.parametrize("options", [o for o in OPTIONS if o != "given"])
def test_parts(evg, oracle_mod, P, sizes, part, options):
    _check(evg, oracle_mod, P, sizes, ("k_update_part", part, 1024), OPTIONS[options])


@pytest.mark.parametrize("P,sizes,part", [p for p in PARTS if p[0] > 16], ids=[f"{p[0]}x{len(p[1])}" for p in PARTS if p[0] > 16])
def test_parts_with_given_gradients(evg, oracle_mod, P, sizes, part):
    _check(evg, oracle_mod, P, sizes, ("k_update_part", part, 1024), dict(given=True))


@pytest.mark.parametrize("P,sizes,part", [(17, [300] * 20, 1), (17, [300] * 60, 2), (17, [300] * 100, 4), (23, [1021] * 80, 4), (10, [1000] * 280, 4)],
                         ids=lambda v: str(v) if not isinstance(v, list) else f"{len(v)}tensors")
@pytest.mark.parametrize("options", [o for o in OPTIONS if o != "given"])
def test_parts_with_messages(evg, oracle_mod, P, sizes, part, options):
    _check(evg, oracle_mod, P, sizes, ("k_update_part", part, 1024), OPTIONS[options], topk_ppm=100_000)


DRAWN = [(5, EDGES * 4, 256), (8, EDGES * 7, 256), (12, EDGES * 5, 256), (6, EDGES + [65_537], 512), (7, EDGES * 20, 512), (16, [265_000, 255], 512), (4, EDGES * 30, 1024)]


@pytest.mark.parametrize("P,sizes,elements", DRAWN, ids=[f"{p[0]}x{len(p[1])}" for p in DRAWN])
@pytest.mark.parametrize("options", ["normal", "norms"])
def test_whole_rings(evg, oracle_mod, P, sizes, elements, options):
    _check(evg, oracle_mod, P, sizes, ("k_update_ring", P, elements), OPTIONS[options])


GIVEN = [(13, EDGES * 5, 256), (16, EDGES * 5, 256), (13, EDGES * 14, 512), (16, EDGES * 14, 512), (11, EDGES * 20, 512), (3, [200, 3] * 210, 256)]


@pytest.mark.parametrize("P,sizes,elements", GIVEN, ids=[f"{p[0]}x{len(p[1])}" for p in GIVEN])
def test_whole_rings_with_given_gradients(evg, oracle_mod, P, sizes, elements):
    _check(evg, oracle_mod, P, sizes, ("k_update_ring", P, elements), dict(given=True))
    _check(evg, oracle_mod, P, sizes, ("k_update_ring", P, elements), dict(given=True, trigger_kind=1, momentum=0.0))


@pytest.mark.parametrize("P,sizes,elements", [(13, [257] * 300 + EDGES, 256), (16, [700] * 240 + EDGES * 4, 256), (9, [1000] * 280, 512)], ids=["13", "16", "9"])
@pytest.mark.parametrize("ppm", [3_000, 400_000])
def test_messages_of_whole_rings_with_given_gradients(evg, oracle_mod, P, sizes, elements, ppm):
    _check(evg, oracle_mod, P, sizes, ("k_update_ring", P, elements), dict(given=True), topk_ppm=ppm)


# whole sends: more than 64 workers, or slices a multiple of 8 KB apart
WALKED = [(9, _on_8k([1300, 7, 515]), 1), (16, _on_8k([9000, 33, 1024]), 1), (64, _on_8k([257, 2, 4097]), 1), (19, _on_8k([1, 3, 8, 2] * 24 + [4097]), 3),
          (65, [1, 3, 8, 2] * 24 + [4097], 5), (23, _on_8k([1, 3, 8, 2] * 49 + [4097]), 6), (66, [1, 3, 8, 2] * 49 + [4097], 9), (17, _on_8k([3] * 640 + [1029]), 17),
          (65, [3] * 640 + [1029], 65)]


@pytest.mark.parametrize("P,sizes,part", WALKED, ids=[f"{p[0]}x{len(p[1])}" for p in WALKED])
@pytest.mark.parametrize("options", list(OPTIONS))
def test_walked_rings(evg, oracle_mod, P, sizes, part, options):
    _check(evg, oracle_mod, P, sizes, ("k_update_walk", part, 0), OPTIONS[options], access_mode=evg.ACCESS_STREAM)


REPLAYED = [p + ("k_update_part", False) for p in PARTS if p[0] > 4] + [p + ("k_update_walk", True) for p in WALKED[2:8]]


@pytest.mark.parametrize("P,sizes,part,which,streams", REPLAYED, ids=[f"{p[3][9:]}{p[0]}x{len(p[1])}" for p in REPLAYED])
@pytest.mark.parametrize("trigger_kind", [0, 1])
def test_replays_that_outlive_an_import(evg, P, sizes, part, which, streams, trigger_kind):
    import torch
    w = _workload(P, sizes, 0, spike_prob=0.3, spike_gain=4.0)
    over = dict(trigger_kind=trigger_kind, access_mode=evg.ACCESS_STREAM if streams else evg.ACCESS_AUTO)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = evg.Ring.from_workload(w, mailbox_fill=0.0, stream=stream, **over)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, **over)
    assert a.update_pass()[:2] == (which, part)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step_next()

    def same(k):
        torch.cuda.synchronize()
        da, db = a.decisions(), b.decisions()
        assert all(np.array_equal(da[key], db[key]) for key in da), k
        for name in ARENAS:
            assert np.array_equal(a.state(name), b.state(name)), (k, name)
    for k in range(3):                     # (the capture itself runs nothing)
        g.replay()
        b.step(k)
        same(k)
    ck = b.export_state()                  # after an odd number of steps
    for k in range(3, 5):
        g.replay()
        b.step(k)
    same(4)
    a.import_state(ck)
    b.import_state(ck)
    for k in range(3, 6):
        g.replay()
        b.step(k)
        same(k)
    a.step(6)                              # on its own stream, which the replays' does not wait for
    b.step(6)
    same(6)
    g.replay()
    b.step(7)
    same(7)
    assert a.stats()["iters"] == b.stats()["iters"] == 8
