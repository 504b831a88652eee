"""The counts of key codes that the update pass of a small cached Top-K ring leaves for the next selection: cleared by all
wavefronts of a workgroup together, so none may add to them before all have done so.  On the CPU the compiled order of clearing,
barrier and additions is read; on the GPU the counts are compared with those of the keys, at windows of one wavefront (the others
have nothing to do and reach their end early), of some and of all, with drawn and given gradients and parts of 1, 2 and 4 workers."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2103_07454_amd import build, inputs

HIST_BINS, COPY, BINS, FIRST_CODE, FINE_BITS = 2048, 256, 128, 64, 17      # of evg_internal.h


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="reads what hipcc compiles")
def test_counts_are_cleared_behind_a_barrier(tmp_path):
    asm = tmp_path / "parts.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "kernels_parts.hip"), "-o", asm],
                   check=True, capture_output=True)
    text = asm.read_text()
    counting = 0
    for m in re.finditer(r"^(_ZN3evg13k_update_part\w+):(.*?)^\.Lfunc_end", text, re.M | re.S):
        order = re.findall(r"^\s+(ds_write_b32|ds_add_u32|s_barrier)\b", m.group(2), re.M)
        if "ds_add_u32" in order:
            counting += 1
            assert order[0] == "ds_write_b32" and "s_barrier" in order[:order.index("ds_add_u32")], (m.group(1), order[:4])
    assert counting == 18          # three gradients, two norms, parts of three sizes


@pytest.mark.gpu
@pytest.mark.parametrize("P,sizes", [(3, [300] * 40 + [257]), (5, [700] * 20), (3, [1000] * 310 + [2049]), (9, [261] * 200),
                                     (12, [1027, 513] * 75)])
@pytest.mark.parametrize("given", [False, True], ids=["drawn", "given"])
def test_counts_are_those_of_the_keys(P, sizes, given):
    import torch
    from paper_2103_07454_amd import evg
    tensors = [inputs.TensorSpec(f"t{i}", (n,), 16 + i % 7, "weight") for i, n in enumerate(sizes)]
    w = inputs.Workload("counts", P, tensors, 0, sigma0=0.05, decay=1.0, seed=P, topk_ppm=100_000, thr_mode=inputs.THR_FIXED, thr_fixed=0.0)
    ring = evg.Ring.from_workload(w, mailbox_fill=0.0, grad_mode=evg.GRAD_BUFFER if given else evg.GRAD_SYNTH)
    grads = [torch.from_numpy(ring.layout.pad(inputs.random_grads(P, w.N, 70 + k, 0.02))).cuda() for k in range(3 if given else 0)]
    starts = np.concatenate([[0], np.cumsum(sizes)])
    for k in range(12):
        ring.step(k, grads[k % 3] if given else None)
        if k < 2:                                            # no Top-K message yet: there is nothing to count about
            continue
        ck = ring.export_state()
        hist = ck["blob"][-P * len(sizes) * HIST_BINS * 4:].view(np.uint32).reshape(P, len(sizes), HIST_BINS)
        anchor = hist[:, :, -1]
        copies = hist.reshape(P, len(sizes), HIST_BINS // COPY, COPY)[..., :BINS + 1].sum(axis=2)
        keys = np.abs(ring.state("x") - ring.state("xhat")).view(np.uint32) >> FINE_BITS
        for l, n in enumerate(sizes):
            if n <= 256:
                continue
            assert (anchor[:, l] != 0xFFFFFFFF).all()
            part = keys[:, starts[l]:starts[l + 1]].astype(np.int64)
            code = np.clip(part - anchor[:, l, None].astype(np.int64), 0, 255) - FIRST_CODE
            for r in range(P):
                c = code[r][code[r] >= 0]
                want = np.bincount(np.minimum(c, BINS), minlength=BINS + 1)
                assert np.array_equal(copies[r, l], want), (k, r, l)
