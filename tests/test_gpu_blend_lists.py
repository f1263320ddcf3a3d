"""The compositing at the edges of its list walk: lists that end inside, at and
just past a 64-entry sub-chunk and a 256-entry round, and the sizes at which a
list is walked in 4, 8 and 32 parts (mean splats per tile of 192 and 1024; at
most 512 and 64 tiles), on images of whole and of ragged tiles.

Image and T_final against the FP32 mirror and every gradient against FP64
autograd, with the bounds of the deep-tile and the needle tests: values within
1e-5 + 8 (k + 2) 2^-24 relative (k splats composited into the pixel), gradients
element by element within 1e-4 |g| + 1e-3 RMS and 1e-4 relative L2.  Pixels with
a decision inside that margin of its threshold are exempt (no upstream
gradient).  The 73,728 splats of the 8-part case are smaller than a pixel, where
the FP32 rounding of a mean (1.5e-5 px at 144) moves alpha by more than the
margin against FP64: their gradients are compared, with the same bounds, with
those of the one-walk route (the same camera on an image of 528 tiles), whose
decisions are the same FP32 ones."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import cpu, ref64
from paper_2407_10707_amd import rga, synth
from tests import helpers

pytestmark = pytest.mark.gpu

CASES = [(1, 32, 32, -1.0), (63, 32, 32, -1.0), (64, 32, 32, -1.0), (65, 31, 29, -1.0),
         (256, 32, 32, -1.0), (257, 32, 32, -1.0), (513, 30, 17, -1.0),     # one walk
         (768, 32, 32, -1.0), (1500, 27, 32, -1.0),                         # 4 parts
         (73_728, 144, 128, -5.6),                                          # 8 parts
         (4096, 32, 32, -1.0), (5000, 17, 31, -1.4)]                        # 32 parts


@pytest.mark.parametrize("n,width,height,scale", CASES)
def test_blend_lists(n, width, height, scale):
    print(f"[blend lists] n={n} {width}x{height}", flush=True)
    rng = np.random.default_rng([31, n])
    cam = synth.default_camera(width, height)
    half = np.array([[1.1 * width / height], [1.1]]) if scale < -2 else np.array([[0.3], [0.3]])
    x = np.concatenate([rng.uniform(-half, half, (2, n)),
                        rng.uniform(-0.2, 0.2, (1, n))]).astype(np.float32)
    A = np.tile(np.eye(3, dtype=np.float32).reshape(9, 1), (1, n))
    q = rng.normal(size=(4, n)).astype(np.float32)
    log_s = rng.normal(scale, 0.2, (3, n)).astype(np.float32)
    opac = rng.uniform(0.005, 0.06, n).astype(np.float32)
    col = rng.random((3, n)).astype(np.float32)
    front = np.ones(n, np.uint8)
    dev = [torch.as_tensor(v).cuda() for v in (x, A, q, log_s, opac, col, front)]
    ws = rga.SplatWorkspace(n, width, height, 12 * n + 1024, "cuda")
    img, T = rga.splat_forward(cam, *dev, ws)
    pre = cpu.splat_preprocess(cam, x, A, q, log_s, opac, front)
    keys, vals, ranges = cpu.splat_bin(cam, pre)
    eimg, eT, margin, napp = cpu.composite_tiles(cam, ranges, vals, pre, opac, col,
                                                 with_applied=True)
    assert ws.count() == len(keys) <= ws.capacity
    gi, gT = img.cpu().numpy(), T.cpu().numpy()
    rel = 1e-5 + 8.0 * (napp + 2) * 2.0 ** -24
    ok = margin > np.maximum(1e-4, rel)
    assert not ((np.abs(gi - eimg) > rel[None] * np.abs(eimg) + 1e-6) & ok[None]).any()
    assert not ((np.abs(gT - eT) > rel * eT) & ok).any()
    w = (rng.uniform(0.5, 1.5, (3, height, width)) * ok[None]).astype(np.float32)
    names = dict(x="dx", quat="dquat", log_s="dlog_s", opac="dopac", color="dcolor")
    if scale < -2:
        big = dataclasses.replace(cam, width=528, height=256)
        wide = np.zeros((3, 256, 528), np.float32)
        wide[:, :height, :width] = w
        ws1 = rga.SplatWorkspace(n, 528, 256, 12 * n + 1024, "cuda")
        img1, _ = rga.splat_forward(big, *dev, ws1)
        g = rga.splat_backward(big, *dev, ws1, img1, torch.as_tensor(wide).cuda())
        ref = {k: g[gk].cpu().numpy() for k, gk in names.items()}
    else:
        p = {k: torch.tensor(v.astype(np.float64), requires_grad=True)
             for k, v in (("x", x), ("quat", q), ("log_s", log_s), ("opac", opac), ("color", col))}
        proj = ref64.project(cam, p["x"], ref64.t64(A), p["quat"], p["log_s"], p["opac"], front)
        img64, _ = ref64.composite(cam, proj, p["opac"], p["color"])
        (img64 * torch.tensor(w.reshape(3, -1).astype(np.float64))).sum().backward()
        ref = {k: p[k].grad.numpy() for k in names}
    # twice: the second backward finds the sums as the first did
    for _ in range(2):
        g = rga.splat_backward(cam, *dev, ws, img, torch.as_tensor(w).cuda())
        for k, gk in names.items():
            helpers.check_grad(k, g[gk].cpu().numpy(), ref[k])
