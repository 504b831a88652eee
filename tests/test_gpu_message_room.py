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
