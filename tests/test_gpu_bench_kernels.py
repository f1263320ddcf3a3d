"""bench.py times and names the shading kernel that a BF16X3 forward ran on: 33,000
Gaussians under 128 directions go to MFMA in one texel per view, and to the FP32 kernel in
two by two."""

import numpy as np
import pytest
import torch

import bench
from oracle import cpu
from paper_2407_10707_amd import rga, synth
from tests import helpers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hv,wv,kernel", [(8, 16, "shade_fwd_bf16x3"), (4, 8, "shade_fwd")])
def test_named_by_what_ran(hv, wv, kernel):
    print(f"[bench kernels] {hv} {wv}", flush=True)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    s = synth.micro_scene(31, 500, 40, 48, he=8, we=16, hv=hv, wv=wv)
    xo, no, _ = cpu.lbs_f32(s["skin"], s["jidx"], s["jw"], s["pos"], s["nrm"])
    _, _, cnt = helpers.oracle_visibility(s)
    pick = np.arange(33_000) % 500
    a = [dev(np.asarray(v)[..., pick]) for v in (xo, no, s["albedo"], s["rough"], s["tint"],
                                                 s["vidx"], s["vw"])]
    a += [dev(cnt), s["kv"], 8, 16, hv, wv, dev(s["env"]), s["cam"].centre.astype(np.float32)]
    t = bench.kernel_times(lambda: rga.shade_gaussians(*a, precision="bf16x3"),
                           ["blend_bwd", "shade_fwd", "shade_fwd_bf16x3"])
    assert list(t) == [kernel]
    assert t[kernel] > 0
