"""Joints in one long chain: 256 of them, one below the other, take no longer than one
thread that walks them in order, forward and back."""

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga

pytestmark = pytest.mark.gpu


def test_chain_of_256():
    """133 us forward and 337 back with one thread, 154 and 264 with the joints' depths by
    a walk through their parents, 60 and 155 now; the fastest of twenty is below 110 and
    230."""
    rng = np.random.default_rng(0)
    dev = lambda a, t: torch.as_tensor(a, dtype=t).cuda()
    th, joints = (dev(rng.normal(0.0, 0.3, (256, 3)), torch.float32) for _ in range(2))
    ds = dev(rng.normal(size=(256, 12)), torch.float32)
    parents = dev(np.arange(256) - 1, torch.int32)
    best = {"pose_skin": 1e9, "pose_skin_bwd": 1e9}
    rga.timing_filter(None)
    rga.timing_enable(True)
    for _ in range(20):
        rga.timing_reset()
        rga.pose_to_skin(th, joints, parents)
        rga.pose_to_skin_backward(th, joints, parents, ds)
        best = {k: min(v, 1e3 * rga.timing_read(k)[0]) for k, v in best.items()}
    rga.timing_enable(False)
    print(f"[pose chain] {best}", flush=True)
    assert best["pose_skin"] < 110
    assert best["pose_skin_bwd"] < 230
