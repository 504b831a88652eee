"""A Top-K ring with a norm pass of its own carries nothing about x from one step to the next: its caller may write
the parameters in between.  Sender and receivers then both go by what was written.  Compared with the oracle, whose
parameters are written alike."""
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


@pytest.mark.parametrize("access", ["stream", "cached"])
@pytest.mark.parametrize("both", [dict(), dict(topk_key=1), dict(trigger_kind=1), dict(xhat_reset=1), dict(delivery_delay=1)],
                         ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()) or "drift")
def test_x_written_between_steps(evg, oracle_mod, both, access):
    import torch
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16, "weight") for i, n in enumerate([3000, 5, 9001, 700])]
    w = inputs.Workload("written", 4, tensors, 9, thr_mode=inputs.THR_FIXED, thr_fixed=0.0, sigma0=0.05, decay=0.9, seed=11,
                        topk_ppm=100_000)
    x0 = inputs.replicate(w.x0(), w.P)
    ring = evg.Ring.from_workload(w, x0, mailbox_fill=float("nan"), norm_mode=evg.NORM_SEPARATE,
                                  access_mode=evg.ACCESS_STREAM if access == "stream" else evg.ACCESS_CACHED, **both)
    orc = oracle_mod.Oracle.from_workload(w, x0, **both)
    rng = np.random.default_rng(7)
    for k in range(w.iters):
        if k in (3, 4, 6):
            x = ring.state("x") + rng.normal(0.0, 0.3, (w.P, w.N)).astype(np.float32)
            ring.x.copy_(torch.from_numpy(ring.layout.pad(x)))
            orc.set_state("x", x)
        torch.cuda.synchronize()
        ring.step(k)
        orc.step(k)
        assert np.array_equal(ring.decisions()["fired"], orc.decisions()["fired"]), k
        for mine, its in zip(ring.message_hashes(), orc.message_hashes()):
            assert np.array_equal(mine, its), k
        for name in ARENAS:
            assert k == 0 or np.array_equal(ring.state(name), orc.state(name)), (k, name)
