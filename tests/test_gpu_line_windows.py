"""Streaming rings cut their tensors so that every sweep of a workgroup begins on a cache line: a
tensor that begins elsewhere gets a first chunk whose leading positions are empty.  Checked against
the oracle with tensors at every such place and of the sizes where the cut can go wrong: as long as
what is left of the first sweep or chunk, one element more or less, and shorter than the lead."""
import pytest

from paper_2103_07454_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def evg():
    from paper_2103_07454_amd import evg as m
    m.lib()
    return m


def _tensors(chunk):
    """Tensors whose lead is 0, 4, 8 .. 28 floats, each in turn as long as `room` allows and one off."""
    out, off = [], 0

    def add(n):
        nonlocal off
        out.append(inputs.TensorSpec(f"t{len(out)}", (n,), 16 + len(out) % 5, "weight"))
        off += (n + 3) // 4 * 4

    for lead in range(4, 32, 4):
        for room in (chunk, 1024, 32):
            for d in (-1, 0, 1):
                while off % 32 != lead:         # short tensors move the next one to its place
                    add(1)
                add(room - lead + d if room - lead + d > 0 else 2)
    return out


@pytest.mark.parametrize("chunk", [1024, 2048, 8192])
@pytest.mark.parametrize("options", [dict(), dict(momentum=0.0), dict(topk_ppm=100_000), dict(topk_ppm=30_000, topk_key=1),
                                     dict(delivery_delay=1), dict(topk_ppm=100_000, delivery_delay=1),
                                     dict(trigger_kind=1), dict(trigger_kind=1, topk_ppm=100_000)],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()) or "whole")
def test_tensors_off_the_lines(evg, oracle_mod, options, chunk):
    from helpers import lockstep
    both = {k: v for k, v in options.items() if k not in ("momentum", "topk_ppm")}
    w = inputs.Workload("lines", 3, _tensors(chunk), 6, momentum=options.get("momentum", 0.9),
                        topk_ppm=options.get("topk_ppm", 0), sigma0=0.05, decay=0.9, seed=chunk)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), chunk_elems=chunk, access_mode=evg.ACCESS_STREAM, **both)
    orc = oracle_mod.Oracle.from_workload(w, x0, **both)
    # the norm-difference trigger subtracts two large norms: decisions must agree, norms only loosely
    differ = "trigger_kind" in both
    rep = lockstep(ring, orc, w.iters, sample_messages=4, norm_rtol=None if differ else 2e-7,
                   norm_abs_of_x=2.5e-7 if differ else None)
    assert rep["rel"]["x"] <= 1e-5 and (differ or all(rep["bitwise"].values())), rep


@pytest.mark.parametrize("topk", [0, 100_000])
def test_saved_state_of_tensors_cut_at_their_start(evg, topk):
    """A blob with fewer sums per tensor, as written where every tensor was cut at its own start, continues alike."""
    import numpy as np
    sizes, chunk, P = [5, 1024, 1020, 3000, 2048, 70], 1024, 3
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16, "weight") for i, n in enumerate(sizes)]
    w = inputs.Workload("blob", P, tensors, 8, sigma0=0.05, decay=0.9, seed=3, topk_ppm=topk)

    def ring():
        return evg.Ring.from_workload(w, mailbox_fill=0.0, chunk_elems=chunk, access_mode=evg.ACCESS_STREAM)

    a, b = ring(), ring()
    for k in range(4):
        a.step(k)
    ck = a.export_state()
    blob = np.array(ck["blob"], dtype=np.uint8)
    offs = np.concatenate([[0], np.cumsum([(n + 3) // 4 * 4 for n in sizes])])[:-1]
    now = [-(-(n + int(o) % 32) // chunk) for n, o in zip(sizes, offs)]
    plain = [-(-n // chunk) for n in sizes]
    assert sum(now) > sum(plain)
    S = P * len(sizes)
    at = 80 + S * (40 + 4 * 1)          # header, then the per-tensor arrays, then the sums of the sweeps
    sums = blob[at:at + 8 * P * sum(now)].view(np.float64).reshape(P, sum(now))
    old, i = np.zeros((P, sum(plain))), 0
    for n, m, j in zip(now, plain, np.concatenate([[0], np.cumsum(plain)])):
        old[:, j] = sums[:, i:i + n].sum(axis=1)
        i += n
    head = blob[:at].copy()
    head[20:24] = np.array([sum(plain)], dtype=np.uint32).view(np.uint8)      # the number of chunks
    rest = blob[at + 8 * P * sum(now):]
    b.import_state(dict(ck, blob=np.concatenate([head, old.reshape(-1).view(np.uint8), rest])))
    for k in range(4, 8):
        a.step(k)
        b.step(k)
    for name in ("x", "xhat", "mbox_l", "mbox_r", "vel"):
        assert np.array_equal(a.state(name), b.state(name)), name
