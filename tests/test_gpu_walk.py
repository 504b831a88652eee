"""Streaming rings are updated by workgroups that walk a window around the ring, in parts where a
network has few windows and many workers.  Checked against the oracle at the ring sizes where the walk
can go wrong: the smallest, around the 64 workers whose marks a wavefront holds at a time, parts of one
worker, and rings whose last part is of one worker or a few."""
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _run(evg, oracle_mod, P, numels, *, norm_mode=0, iters=7, **kw):
    from helpers import lockstep
    both = {k: kw.pop(k) for k in ("trigger_kind", "topk_key", "xhat_reset") if k in kw}
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate(numels)]
    w = inputs.Workload("walk", P, tensors, iters, sigma0=0.05, decay=0.9, seed=P, **kw)
    x0 = inputs.replicate(w.x0(), P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), access_mode=evg.ACCESS_STREAM, norm_mode=norm_mode, **both)
    orc = oracle_mod.Oracle.from_workload(w, x0, **both)
    differ = "trigger_kind" in both
    rep = lockstep(ring, orc, w.iters, sample_messages=8, norm_rtol=None if differ else 2e-7,
                   norm_abs_of_x=2.5e-7 if differ else None)
    assert rep["rel"]["x"] <= 1e-5 and (differ or all(rep["bitwise"].values())), rep


# so few windows: 3 and 4 workers in one part, more in parts of one worker (whole sends of at most 64 workers are not walked, nor further down: those
# that are, test_gpu_passes.py)
@pytest.mark.parametrize("P", [3, 4, 15, 16, 17, 23, 63, 64, 65, 66, 130])
@pytest.mark.parametrize("kw", [dict(), dict(momentum=0.0, spike_prob=0.3, spike_gain=4.0), dict(topk_ppm=100_000),
                                dict(topk_ppm=20_000, dist=1, topk_key=1)], ids=["whole", "plain", "topk", "topk_value"])
def test_ring_sizes(evg, oracle_mod, P, kw):
    _run(evg, oracle_mod, P, [1300, 7, 2048, 515], **kw)


# more than 600 windows: one part whatever the number of workers
@pytest.mark.parametrize("P", [16, 64, 65])
@pytest.mark.parametrize("topk", [0, 100_000])
def test_whole_ring(evg, oracle_mod, P, topk):
    _run(evg, oracle_mod, P, [3] * 640 + [1029], topk_ppm=topk, iters=4)


@pytest.mark.parametrize("P", [5, 18])
@pytest.mark.parametrize("topk", [0, 100_000])
@pytest.mark.parametrize("norm_mode,trigger_kind", [(1, 0), (0, 1), (1, 1)])
def test_norms(evg, oracle_mod, P, topk, norm_mode, trigger_kind):
    kw = dict(trigger_kind=1) if trigger_kind else {}
    _run(evg, oracle_mod, P, [9000, 33, 1024], topk_ppm=topk, norm_mode=norm_mode, **kw)


# A selection's last bins are 64 where the threshold was expected, 1024 where it moved by octaves, 512 in rings whose norms are a pass of
# their own; chunks that end with a load of sixteen codes, within one, and after the first of a lane's two
@pytest.mark.parametrize("numels", [[8192, 4096, 4112, 15], [8208, 4097, 16, 12_289]], ids=["whole", "ragged"])
@pytest.mark.parametrize("kw", [dict(), dict(spike_prob=0.5, spike_gain=50.0), dict(norm_mode=1), dict(topk_key=1)],
                         ids=["expected", "moved", "plain", "value"])
def test_last_bins_and_codes(evg, oracle_mod, numels, kw):
    _run(evg, oracle_mod, 5, numels, topk_ppm=50_000, iters=9, **kw)


# Tensors of one window each, and a longer one.  Of about 100 windows Top-K goes in parts of 3 workers (19 = 6 * 3 + 1), 9 (65),
# 17 (130), whole sends of 5 (65) and 9 (130); of 200 Top-K of 4 (16), 12 (23), both of 9 (66); of 330 Top-K in one part (15), of 9 (17), both of 10 (65).
@pytest.mark.parametrize("windows,P", [(100, 19), (100, 65), (100, 130), (200, 16), (200, 23), (200, 66), (330, 15), (330, 17), (330, 65)])
@pytest.mark.parametrize("kw", [dict(), dict(topk_ppm=100_000)], ids=["whole", "topk"])
def test_parts(evg, oracle_mod, windows, P, kw):
    _run(evg, oracle_mod, P, [1, 3, 8, 2] * ((windows - 5) // 4) + [4097], iters=5, **kw)


# xhat reset at events: the walk reads the mailboxes (one part: up to 5 workers, or more than 600 windows; parts: no walk)
@pytest.mark.parametrize("P,numels", [(3, [1300, 7, 2048, 515]), (5, [9000, 33, 1024]), (4, [20480, 3]), (16, [3] * 640 + [1029]),
                                      (66, [2] * 620 + [700]), (17, [1300, 7])], ids=["3", "5", "chunks", "16", "66", "parts"])
@pytest.mark.parametrize("kw", [dict(topk_ppm=100_000), dict(topk_ppm=20_000, dist=1, topk_key=1, momentum=0.0),
                                dict(topk_ppm=300_000, trigger_kind=1, spike_prob=0.3, spike_gain=4.0), dict(topk_ppm=100_000, norm_mode=1)],
                         ids=["drift", "value", "norms", "separate"])
def test_xhat_reset(evg, oracle_mod, P, numels, kw):
    _run(evg, oracle_mod, P, numels, iters=6, xhat_reset=1, **kw)


@pytest.mark.parametrize("chunk", [1024, 8192])
def test_xhat_reset_with_given_gradients(evg, oracle_mod, chunk):
    import torch
    from helpers import lockstep
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i, "weight") for i, n in enumerate([9000, 5, 4097])]
    w = inputs.Workload("walk", 4, tensors, 7, seed=4, topk_ppm=100_000)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), access_mode=evg.ACCESS_STREAM, xhat_reset=1, grad_mode=1,
                                  chunk_elems=chunk)
    orc = oracle_mod.Oracle.from_workload(w, x0, xhat_reset=1, grad_mode=1)
    given = {k: inputs.random_grads(w.P, w.N, 900 + k, 0.02) for k in range(w.iters)}
    on_gpu = {k: torch.from_numpy(ring.layout.pad(g)).cuda() for k, g in given.items()}
    rep = lockstep(ring, orc, w.iters, grads=given.get, gpu_grads=on_gpu.get, sample_messages=8)
    assert all(rep["bitwise"].values()), rep
