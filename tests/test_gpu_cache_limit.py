"""Top-K rings that are larger than the last-level cache are streamed, also where cached accesses are asked for: no copies
of the parameters are kept for them, and they run as fast as streaming ones.  Checked on both sides of the limit (seven arenas, 256
MB) against the ring with streaming accesses, bit for bit."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

P, LIMIT = 8, (256 << 20) // (7 * 8 * 4) // 64 * 64        # elements a worker


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


@pytest.mark.parametrize("topk", [0, 100_000])
@pytest.mark.parametrize("beyond", [0, 64])
def test_cached_accesses_are_asked_for(evg, topk, beyond):
    n = LIMIT + beyond
    tensors = [inputs.TensorSpec("a", (1000,), 16, "weight"), inputs.TensorSpec("b", (n - 1000 - 8,), 16, "weight"),
               inputs.TensorSpec("c", (7,), 16, "weight")]
    w = inputs.Workload("limit", P, tensors, 6, sigma0=0.05, decay=0.9, seed=9, topk_ppm=topk)
    a = evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=evg.ACCESS_CACHED, chunk_elems=8192)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, access_mode=evg.ACCESS_STREAM, chunk_elems=8192)
    for k in range(w.iters):
        a.step(k)
        b.step(k)
        assert np.array_equal(a.decisions()["fired"], b.decisions()["fired"])
    for name in ("x", "xhat", "vel", "mbox_l", "mbox_r"):
        assert a.torch.equal(getattr(a, name), getattr(b, name)), name
    copies = a.stats()["library_bytes"] - b.stats()["library_bytes"] > P * a.layout.npad * 4
    assert copies == (not topk or beyond == 0)


# (elements a worker, workers, seven arenas fit the cache, the ring is cached): fewer and more than 600 pieces, and on both sides of
# the limits of 256 MB for seven arenas and 220 MB for five
@pytest.mark.parametrize("n,P,fit,cached", [(112_000, 64, True, True), (150_004, 64, False, True), (182_000, 64, False, False),
                                            (700_001, 10, True, False)])
@pytest.mark.parametrize("over", [dict(), dict(xhat_reset=1), dict(norm_mode=1)], ids=["", "reset", "separate"])
def test_rings_of_few_windows(evg, n, P, fit, cached, over):
    tensors = [inputs.TensorSpec("a", (1000,), 16, "weight"), inputs.TensorSpec("b", (n - 1008,), 16, "weight"),
               inputs.TensorSpec("c", (7,), 16, "weight")]
    w = inputs.Workload("few", P, tensors, 6, sigma0=0.05, decay=0.9, seed=9, topk_ppm=50_000)
    x0 = inputs.replicate(w.x0(), P)
    a = evg.Ring.from_workload(w, x0, mailbox_fill=0.0, **over)
    b = evg.Ring.from_workload(w, x0, mailbox_fill=0.0, access_mode=evg.ACCESS_STREAM, **over)
    a.timing(True)
    for k in range(w.iters):
        a.step(k)
        b.step(k)
        assert np.array_equal(a.decisions()["fired"], b.decisions()["fired"])
        for mine, its in zip(a.message_hashes(), b.message_hashes()):
            assert np.array_equal(mine, its), k
    for name in ("x", "xhat", "vel", "mbox_l", "mbox_r"):
        assert a.torch.equal(getattr(a, name), getattr(b, name)), name
    copies = a.stats()["library_bytes"] - b.stats()["library_bytes"] > P * a.layout.npad * 4
    assert copies == (cached and fit and not over)
    if cached and not copies:                      # the messages go into the mailboxes ahead of the update pass
        assert a.timing_read()["topk_send"][1] == w.iters
