"""Cached Top-K rings whose tensors are not too long: one workgroup per tensor makes the whole selection, from the key codes and
counts that the update pass leaves (a pass in parts of the ring).  Checked against the oracle, message by message, at the
sizes where it can go wrong: tensors of a wavefront (up to 256 elements) and one more, ends of groups of 256, of the codes that a
workgroup holds at once (163 840), twice as many and the longest it takes (819 200); parts of 1, 2 and 4 workers, closed rings and last parts of
one; thresholds that leave the counted codes (spikes, decay), ties, and blobs that move to and from streaming rings."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

ARENAS = ("x", "xhat", "vel", "mbox_l", "mbox_r")


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _workload(P, sizes, iters, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate(sizes)]
    base = dict(sigma0=0.05, decay=0.95, seed=P, topk_ppm=100_000)
    base.update(kw)
    return inputs.Workload("choose", P, tensors, iters, **base)


def _run(evg, oracle_mod, w, **both):
    from helpers import lockstep
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), **both)
    orc = oracle_mod.Oracle.from_workload(w, x0, **both)
    differ = "trigger_kind" in both
    rep = lockstep(ring, orc, w.iters, sample_messages=8, norm_rtol=None if differ else 2e-7, norm_abs_of_x=2.5e-7 if differ else None)
    assert rep["rel"]["x"] <= 1e-5 and (differ or all(rep["bitwise"].values())), rep


@pytest.mark.parametrize("sizes", [[1, 2, 3, 5, 255, 256, 257, 258], [1023, 1024, 1025, 2047, 2049], [16_383, 16_385], [163_839, 4],
                                   [163_841], [327_680, 7], [327_681, 260]], ids=lambda s: "_".join(map(str, s)))
@pytest.mark.parametrize("kw", [dict(), dict(topk_ppm=7_000, dist=1, topk_key=1)], ids=["drift", "value"])
def test_sizes(evg, oracle_mod, sizes, kw):
    kw = dict(kw)
    both = dict(topk_key=kw.pop("topk_key")) if "topk_key" in kw else {}
    _run(evg, oracle_mod, _workload(3, sizes, 6, **kw), **both)


# streaming rings stage by codes, sixteen to a lane: ends of those, of their words, of groups of 256 and of chunks; tensors begin anywhere
# on their cache line (every other tensor is of odd length)
@pytest.mark.parametrize("chunk", [1024, 2048, 4096, 8192])
@pytest.mark.parametrize("topk_key", [0, 1])
def test_streamed_sizes(evg, oracle_mod, chunk, topk_key):
    from helpers import lockstep
    sizes = [15, 16, 17, 31, 33, 1, 241, 255, 257, 1009, 1024, 1039, 4095, 4097, 8175, 8191, 8209, 16_385, 24_575]
    w = _workload(3, sizes, 6, topk_ppm=20_000)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), topk_key=topk_key, access_mode=evg.ACCESS_STREAM, chunk_elems=chunk)
    orc = oracle_mod.Oracle.from_workload(w, x0, topk_key=topk_key)
    rep = lockstep(ring, orc, w.iters, sample_messages=8)
    assert all(rep["bitwise"].values()), rep


# few windows: parts of one worker; some 1000 of a window and worker: of two; more: of four
@pytest.mark.parametrize("P,sizes", [(3, [700] * 3), (5, [300] * 4), (3, [1021] * 310), (11, [259] * 90), (4, [300] * 401),
                                     (9, [261] * 200), (12, [1027] * 150)])
@pytest.mark.parametrize("kw", [dict(spike_prob=0.3, spike_gain=9.0), dict(momentum=0.0, decay=0.3), dict(trigger_kind=1), dict(gradients=True)],
                         ids=["spikes", "decay_plain", "norms", "given"])
def test_parts(evg, oracle_mod, P, sizes, kw):
    import torch
    from helpers import lockstep
    kw = dict(kw)
    if kw.pop("gradients", False):
        w = _workload(P, sizes, 6)
        x0 = inputs.replicate(w.x0(), P)
        ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), grad_mode=1)
        orc = oracle_mod.Oracle.from_workload(w, x0, grad_mode=1)
        given = {k: inputs.random_grads(P, w.N, 900 + k, 0.02) for k in range(w.iters)}
        on_gpu = {k: torch.from_numpy(ring.layout.pad(g)).cuda() for k, g in given.items()}
        rep = lockstep(ring, orc, w.iters, grads=given.get, gpu_grads=on_gpu.get, sample_messages=8)
        assert all(rep["bitwise"].values()), rep
        return
    both = dict(trigger_kind=kw.pop("trigger_kind")) if "trigger_kind" in kw else {}
    _run(evg, oracle_mod, _workload(P, sizes, 7, **kw), **both)


@pytest.mark.parametrize("sizes", [[100, 3000, 20_000], [20_480]])
def test_ties_that_do_not_all_win(evg, oracle_mod, sizes):
    """Gradients of a few values: from some tens to thousands of keys equal the threshold."""
    import torch
    from helpers import lockstep
    w = _workload(4, sizes, 10, thr_mode=inputs.THR_FIXED, thr_fixed=0.0)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, grad_mode=1, lr=0.5, momentum=0.0)
    orc = oracle_mod.Oracle.from_workload(w, x0, grad_mode=1, lr=0.5, momentum=0.0)
    given = {}
    for k in range(w.iters):
        g = np.round(inputs.random_grads(w.P, w.N, 40 + k) * (200.0 if k % 2 else 2.0)) * np.float32(0.25)
        given[k] = g.astype(np.float32)
    on_gpu = {k: torch.from_numpy(ring.layout.pad(g)).cuda() for k, g in given.items()}
    rep = lockstep(ring, orc, w.iters, grads=given.get, gpu_grads=on_gpu.get, sample_messages=12)
    assert all(rep["bitwise"].values()), rep


@pytest.mark.parametrize("written_by", ["stream", "cached"])
def test_blobs_between_streaming_and_cached_rings(evg, written_by):
    w = _workload(5, [40_000, 300, 7, 2049], 12, spike_prob=0.2, spike_gain=3.0)
    modes = dict(stream=evg.ACCESS_STREAM, cached=evg.ACCESS_CACHED)
    a = evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=modes[written_by])
    for k in range(5):
        a.step(k)
    ck = a.export_state()
    rings = [evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=m) for m in modes.values()]
    for r in rings:
        r.import_state(ck)
    again = evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=modes[written_by])
    again.import_state(rings[0].export_state())
    for k in range(5, 12):
        for r in [a, again] + rings:
            r.step(k)
        for r in [again] + rings:
            assert np.array_equal(a.decisions()["fired"], r.decisions()["fired"]), k
            for mine, its in zip(a.message_hashes(), r.message_hashes()):
                assert np.array_equal(mine, its), k
    for r in [again] + rings:
        for name in ARENAS:
            assert np.array_equal(a.state(name), r.state(name)), name


def _not_staged(evg, oracle_mod, sizes, P, iters, given=None, **kw):
    """What evg_stats counts in each iteration of a run that agrees with the oracle: chunks of tensors of more than 256 elements whose
    selection read all keys instead of going by codes."""
    import torch
    w = _workload(P, sizes, iters, decay=1.0, thr_mode=inputs.THR_FIXED, thr_fixed=0.0, **kw)
    x0 = inputs.replicate(w.x0(), P)
    more = dict(grad_mode=1, lr=0.5, momentum=0.0) if given is not None else {}
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=0.0, **more)
    orc = oracle_mod.Oracle.from_workload(w, x0, **more)
    counts = [0]
    for k in range(iters):
        g = None if given is None else given(k, w.N)
        ring.step(k, None if g is None else torch.from_numpy(ring.layout.pad(g)).cuda())
        orc.step(k, grad=g)
        counts.append(ring.stats()["chunks_not_staged"])
        for mine, its in zip(ring.message_hashes(), orc.message_hashes()):
            assert np.array_equal(mine, its), k
    for name in ("x", "xhat"):
        assert np.array_equal(ring.state(name), orc.state(name)), name
    return np.diff(counts)


@pytest.mark.parametrize("sizes,kw", [([300, 4000, 20_000, 100_000], dict(momentum=0.0)), ([257, 320_000], dict(topk_ppm=10_000)),
                                      ([256, 17], dict())], ids=["small", "longest", "wavefront"])
def test_selections_go_by_codes(evg, oracle_mod, sizes, kw):
    """Only a tensor's first Top-K message is told from all of its keys; later ones go by the codes and counts of the update pass."""
    n = _not_staged(evg, oracle_mod, sizes, 3, 10, **kw)
    chunks = 3 * sum(-(-s // 2048) for s in sizes if s > 256)
    assert n.tolist() == [0, chunks] + [0] * 8


# Drifts of one size: in half of the elements, more keys than the list holds have the threshold's code, and all keys are read; in a
# twentieth, and with a share below that, more ties than a wavefront sorts out, from the codes all the same
@pytest.mark.parametrize("every,ppm,lists", [(2, 100_000, False), (20, 20_000, True)])
def test_more_keys_of_a_code_than_the_list_holds(evg, oracle_mod, every, ppm, lists):
    sizes = [30_000]

    def given(k, N):
        g = inputs.random_grads(3, N, 70 + k, 1e-3)
        g[:, (7 * k) % every::every] = 64.0
        return g
    n = _not_staged(evg, oracle_mod, sizes, 3, 8, given, topk_ppm=ppm)
    assert n[:2].tolist() == [0, 45] and ((n[3:] == 0).all() if lists else (n[3:] > 0).any()), n


@pytest.mark.parametrize("P,n", [(3, 655_360), (3, 655_361), (4, 819_200), (4, 819_201)])
def test_the_longest_tensors_of_a_workgroup(evg, oracle_mod, P, n):
    _run(evg, oracle_mod, _workload(P, [n, 9], 4, topk_ppm=30_000))


# a spike drives a long tensor's threshold out of its codes; with spikes only shorter ones are one workgroup's, and with those the ring's update pass
@pytest.mark.parametrize("n,spikes,want", [(327_680, 0.1, "k_update_ring"), (327_681, 0.1, "k_update"), (327_681, 0.0, "k_update_ring")])
def test_long_tensors_with_spikes_are_not_one_workgroups(evg, oracle_mod, n, spikes, want):
    w = _workload(6, [n, 9], 4, topk_ppm=30_000, spike_prob=spikes, spike_gain=5.0)
    assert evg.Ring.from_workload(w).update_pass()[0] == want
    _run(evg, oracle_mod, w)
