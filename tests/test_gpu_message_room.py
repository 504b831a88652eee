"""A Top-K message never grows past its K entries.  A ring whose update pass carries the histograms of the next
selection finds other numbers of winners if its caller writes the parameters of a tensor between two steps.  Nothing
is then sent of that tensor in that iteration, and the messages of all other tensors, which lie next to its own,
stay what they were."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


# streaming: the whole ring, and in parts of 8 workers; cached; messages applied ahead of the update; delayed
@pytest.mark.parametrize("P,over", [(4, dict(access_mode=1)), (17, dict(access_mode=1)), (4, dict(access_mode=2)),
                                    (4, dict(access_mode=2, xhat_reset=1)), (4, dict(access_mode=1, delivery_delay=1))],
                         ids=["stream", "parts", "cached", "reset", "delay"])
def test_other_tensors_messages_stay(evg, P, over):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16, "weight") for i, n in enumerate([3000, 40, 9001, 700])]
    w = inputs.Workload("room", P, tensors, 8, thr_mode=inputs.THR_FIXED, thr_fixed=0.0, sigma0=0.05, decay=0.9, seed=5,
                        topk_ppm=100_000)
    a, b = evg.Ring.from_workload(w, mailbox_fill=0.0, **over), evg.Ring.from_workload(w, mailbox_fill=0.0, **over)
    for k in range(3):
        a.step(k)
        b.step(k)
    written, start = 2, int(a.layout.offsets[2])
    b.x[:, start:start + 9001] *= 1000.0           # every key lies above the bin the histogram names
    for k in range(3, 6):
        a.step(k)
        b.step(k)
        assert (b.decisions()["fired"] == 2).all()
        for r in range(P):
            for l in range(w.L):
                ia, va = a.message(r, l)
                ib, vb = b.message(r, l)
                assert ib.size == (0 if l == written and k == 3 else ia.size) and ia.size > 0
                if l == written:
                    assert (np.diff(ib.astype(np.int64)) > 0).all()
                else:
                    assert np.array_equal(ia, ib) and np.array_equal(va, vb), (k, r, l)
        idx, _ = b.message_hashes()
        assert ((idx[:, written] == 0) == (k == 3)).all()
    if not over.get("xhat_reset"):                 # what the neighbours hold is what was sent
        assert np.array_equal(b.state("mbox_l"), np.roll(b.state("xhat"), 1, axis=0))
        assert np.array_equal(b.state("mbox_r"), np.roll(b.state("xhat"), -1, axis=0))
    for name in ("x", "xhat", "mbox_l", "mbox_r", "vel"):
        sa, sb = a.state(name), b.state(name)
        for l, (n, o) in enumerate(zip([3000, 40, 9001, 700], [0, 3000, 3040, 12041])):
            assert l == written or np.array_equal(sa[:, o:o + n], sb[:, o:o + n]), (name, l)


# A write that moves a few keys from below the threshold to above it, or the other way round, leaves all counts of keys with K winners.  What
# is sent all the same is what the message says: the groups of 256 elements in which another number wins send nothing.
@pytest.mark.parametrize("up", [True, False], ids=["to_above", "to_below"])
@pytest.mark.parametrize("P,over", [(4, dict(access_mode=1)), (17, dict(access_mode=1)), (4, dict(access_mode=1, xhat_reset=1)),
                                    (17, dict(access_mode=1, xhat_reset=1)), (4, dict(access_mode=1, delivery_delay=1)),
                                    (4, dict(access_mode=2)), (12, dict(access_mode=2))],
                         ids=["stream", "parts", "reset", "reset_ahead", "delay", "cached", "cached_parts"])
def test_a_message_is_what_its_sender_and_its_receivers_take(evg, P, over, up):
    import torch
    sizes = [3000, 40, 9001, 700] + ([1024 * 24] * 5 if over["access_mode"] == 2 and P > 4 else [])
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16, "weight") for i, n in enumerate(sizes)]
    w = inputs.Workload("room", P, tensors, 8, thr_mode=inputs.THR_FIXED, thr_fixed=0.0, sigma0=0.05, decay=0.9, seed=6, topk_ppm=100_000)
    ring = evg.Ring.from_workload(w, mailbox_fill=0.0, **over)
    starts = np.concatenate([[0], np.cumsum(sizes)])
    for k in range(4):
        ring.step(k)
    for k in range(4, 7):
        x, before = ring.state("x"), {name: ring.state(name) for name in ("xhat", "mbox_l", "mbox_r")}
        moved = np.zeros((P, w.N), bool)
        if k == 4:
            for l in (0, 2):
                part = slice(int(starts[l]), int(starts[l + 1]))
                order = np.argsort(np.abs(x[:, part] - before["xhat"][:, part]), axis=1, kind="stable")
                some = (order[:, :5] if up else order[:, -5:]) + starts[l]
                np.put_along_axis(x, some, np.take_along_axis(before["xhat"], some, axis=1) + np.float32(50.0 if up else 0.0), axis=1)
                np.put_along_axis(moved, some, True, axis=1)
            ring.x.copy_(torch.from_numpy(ring.layout.pad(x)))
            torch.cuda.synchronize()
        ring.step(k)
        assert (ring.decisions()["fired"] == 2).all()
        after = {name: ring.state(name) for name in ("xhat", "mbox_l", "mbox_r")}
        hashes = ring.message_hashes()[0]
        for r in range(P):
            sent = np.zeros(w.N, bool)
            for l, n in enumerate(sizes):
                idx, val = ring.message(r, l)
                K, lead = -(-n // 10), int(ring.layout.offsets[l]) % 32 if over["access_mode"] == 1 else 0
                if k == 4 and l in (0, 2):
                    groups = set((np.nonzero(moved[r, starts[l]:starts[l + 1]])[0] + lead) // 256)
                    assert 0 < idx.size < K and not groups & set((idx + lead) // 256), (k, r, l)
                else:
                    assert idx.size == K, (k, r, l)
                assert (np.diff(idx.astype(np.int64)) > 0).all() and idx[-1] < n, (k, r, l)
                assert np.array_equal(val, x[r, starts[l] + idx]) and hashes[r, l] == _index_hash(idx), (k, r, l)
                sent[starts[l] + idx] = True
            for name, whose in (("xhat", r), ("mbox_l", (r + 1) % P), ("mbox_r", (r - 1) % P)):
                # (cached rings: in the step after the write a neighbour takes what the copies of x held for it)
                if over["access_mode"] == 2 and name != "xhat":
                    continue
                want = before[name][whose].copy()
                want[sent] = x[r, sent]
                if name == "xhat" and over.get("xhat_reset"):
                    want = x[r]
                assert np.array_equal(after[name][whose], want), (k, r, name)


def _index_hash(idx):
    """The index half of evg_message_hashes: the sum of SplitMix64's finaliser over the indices."""
    with np.errstate(over="ignore"):
        z = idx.astype(np.uint64) + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ z >> np.uint64(30)) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ z >> np.uint64(27)) * np.uint64(0x94D049BB133111EB)
        return (z ^ z >> np.uint64(31)).sum(dtype=np.uint64)
