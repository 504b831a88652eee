"""State blobs move between the rings of one configuration however their tensors are cut into chunks: streaming
rings cut them on cache lines, cached rings at the tensors' own starts.  The continued run is compared bit for bit
with the ring that wrote the blob."""
import numpy as np
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu

ARENAS = ("x", "xhat", "mbox_l", "mbox_r", "vel")


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _workload(sizes, **kw):
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16, "weight") for i, n in enumerate(sizes)]
    return inputs.Workload("saved", 3, tensors, 10, sigma0=0.05, decay=0.9, seed=3, **kw)


def _chunks(sizes, chunk, on_lines):
    offs = np.concatenate([[0], np.cumsum([(n + 3) // 4 * 4 for n in sizes])])[:-1]
    return [-(-(n + (int(o) % 32 if on_lines else 0)) // chunk) for n, o in zip(sizes, offs)]


def _same_run(a, b, first, last):
    for k in range(first, last):
        a.step(k)
        b.step(k)
        da, db = a.decisions(), b.decisions()
        assert np.array_equal(da["fired"], db["fired"]), k
        # the sums of a tensor are added in another order
        np.testing.assert_allclose(da["norm"], db["norm"], rtol=2e-7, atol=1e-37)
    for name in ARENAS:
        assert np.array_equal(a.state(name), b.state(name)), name


# tensors that take a chunk more on cache lines
@pytest.mark.parametrize("sizes,chunk", [([4, 2048], 2048), ([5, 1024, 1020, 3000, 2048, 70], 1024), ([8, 8190, 4, 16380], 8192)])
@pytest.mark.parametrize("kw", [dict(), dict(topk_ppm=100_000), dict(trigger_kind=1), dict(trigger_kind=1, topk_ppm=100_000)],
                         ids=["whole", "topk", "norms", "norms_topk"])
@pytest.mark.parametrize("written_by", ["stream", "cached"])
def test_between_access_modes(evg, sizes, chunk, kw, written_by):
    assert sum(_chunks(sizes, chunk, True)) > sum(_chunks(sizes, chunk, False))
    kw = dict(kw)
    over = dict(trigger_kind=kw.pop("trigger_kind")) if "trigger_kind" in kw else {}
    w = _workload(sizes, **kw)
    modes = dict(stream=evg.ACCESS_STREAM, cached=evg.ACCESS_CACHED)

    def ring(mode):
        return evg.Ring.from_workload(w, mailbox_fill=0.0, chunk_elems=chunk, access_mode=modes[mode], **over)

    a, b = ring(written_by), ring("cached" if written_by == "stream" else "stream")
    for k in range(4):
        a.step(k)
    b.import_state(a.export_state())
    _same_run(a, b, 4, 10)


# its tensors take as many chunks as the other ring's would on cache lines, more, or fewer
@pytest.mark.parametrize("sizes", [[4, 2052], [4, 4097], [4, 2048, 1], [2048]], ids=str)
def test_a_blob_of_other_tensors_is_refused(evg, sizes):
    a = evg.Ring.from_workload(_workload(sizes), chunk_elems=2048, access_mode=evg.ACCESS_CACHED)
    b = evg.Ring.from_workload(_workload([4, 2048]), chunk_elems=2048, access_mode=evg.ACCESS_CACHED)
    ck = dict(a.export_state(), **{name: b.export_state()[name] for name in ARENAS})
    with pytest.raises(evg.EvgError) as e:
        b.import_state(ck)
    assert e.value.status == 1


# version 3: tensors cut at their own starts, and four words where later versions have one
@pytest.mark.parametrize("access", ["stream", "cached"])
@pytest.mark.parametrize("kw", [dict(), dict(topk_ppm=100_000), dict(trigger_kind=1, topk_ppm=100_000)], ids=["whole", "topk", "norms_topk"])
def test_blobs_of_version_3_are_read(evg, kw, access):
    sizes, chunk, P = [5, 1024, 1020, 3000, 2048, 70], 1024, 3
    kw = dict(kw)
    over = dict(trigger_kind=kw.pop("trigger_kind")) if "trigger_kind" in kw else {}
    w = _workload(sizes, **kw)
    a = evg.Ring.from_workload(w, mailbox_fill=0.0, chunk_elems=chunk, access_mode=evg.ACCESS_CACHED, **over)
    b = evg.Ring.from_workload(w, mailbox_fill=0.0, chunk_elems=chunk,
                               access_mode=evg.ACCESS_STREAM if access == "stream" else evg.ACCESS_CACHED, **over)
    for k in range(4):
        a.step(k)
    ck = a.export_state()
    # header, the per-tensor arrays, one sum per sweep, the iteration
    at = 80 + P * len(sizes) * (40 + 4) + 8 * P * sum(_chunks(sizes, chunk, False)) + 32
    old = np.insert(np.array(ck["blob"], dtype=np.uint8), at, np.full(12, 7, np.uint8))
    old[8:12] = np.array([3], np.uint32).view(np.uint8)
    b.import_state(dict(ck, blob=old))
    assert a.stats()["chunks_not_staged"] == b.stats()["chunks_not_staged"]
    _same_run(a, b, 4, 10)


@pytest.mark.parametrize("topk", [0, 100_000])
def test_steps_on_a_stream_of_their_own_follow_an_import(evg, topk):
    """The import is over when it returns, for a stream that waits for no other: the copies of x that cached rings
    send from are those of the imported parameters."""
    import torch
    w = _workload([700_003, 60_000, 5], topk_ppm=topk)
    a = evg.Ring.from_workload(w, mailbox_fill=0.0)
    for k in range(4):
        a.step(k)
    ck = a.export_state()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b = evg.Ring.from_workload(w, mailbox_fill=0.0, stream=s)
        b.step(0)
        b.import_state(ck)
        b.step(4)
        b.step_next()
    s.synchronize()
    a.step(4)
    a.step(5)
    _same_run(a, b, 6, 8)
