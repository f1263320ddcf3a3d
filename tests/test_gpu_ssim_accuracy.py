"""Accuracy of the image loss's gradient where the variances cancel: its error
against the FP64 oracle is no larger than that of the formula itself in FP32, with
x^2 and y^2 filtered apart and the same order of operations (numpy, fused
multiply-adds as float32(a b + c) from float64).  The two differ by the rounding of
a division only, less than one per cent of the error, so the limit is 1.03 times
(one map of x^2 + y^2 in the place of the two: 1.08 to 1.6 times)."""

import numpy as np
import pytest
import torch

from oracle import ref64
from paper_2407_10707_amd import rga

pytestmark = pytest.mark.gpu

F = np.float32


def _blur(v):
    g = ref64.ssim_window().numpy().astype(F).astype(np.float64)
    H, W = v.shape
    for axis, n in ((1, W), (0, H)):
        pad = np.pad(v, [(5, 5) if a == axis else (0, 0) for a in (0, 1)])
        s = np.zeros((H, W), F)
        for j in range(11):
            tap = pad[:, j:j + n] if axis else pad[j:j + n]
            s = (g[j] * tap.astype(np.float64) + s).astype(F)
        v = s
    return v


def _gradient32(x, y):
    """dS/dx, the gradient of the sum of the SSIM map."""
    mx, my = _blur(x), _blur(y)
    sxx, syy, sxy = _blur(x * x) - mx * mx, _blur(y * y) - my * my, _blur(x * y) - mx * my
    c1, c2 = F(1e-4), F(9e-4)
    a1, a2 = F(2) * mx * my + c1, F(2) * sxy + c2
    b1, b2 = mx * mx + my * my + c1, sxx + syy + c2
    inv = F(1) / (b1 * b2)
    s = a1 * a2 * inv
    dmu = F(2) * my * a2 * inv - F(2) * mx * s * (inv * b2)
    dsx, dsxy = -s * (inv * b1), F(2) * a1 * inv
    ga, gb, gc = _blur(dmu - F(2) * mx * dsx - my * dsxy), _blur(dsx), _blur(dsxy)
    return ga + F(2) * x * gb + y * gc


def _images(kind, seed, H, W):
    r = np.random.default_rng(seed)
    coarse = torch.tensor(r.random((1, 1, H // 16 + 2, W // 16 + 2)))
    smooth = torch.nn.functional.interpolate(coarse, size=(H, W), mode="bilinear")[0, 0].numpy()
    off = lambda v, s: np.clip(v + s * r.standard_normal((H, W)), 0, 1)
    if kind == "flat":
        x, y = np.full((H, W), 0.7), off(np.full((H, W), 0.3), 0.002)
    elif kind == "smooth":
        x, y = smooth, off(smooth, 0.05)
    else:
        y = off(smooth, 0.05 if kind == "textured" else 0.0)
        x = off(y, 0.05 if kind == "textured" else 0.01)
    return x.astype(F), y.astype(F)


@pytest.mark.parametrize("kind", ["textured", "smooth", "close", "flat"])
@pytest.mark.parametrize("seed", [1, 2])
def test_gradient_error(kind, seed):
    H, W = 300, 277
    print(f"[ssim accuracy] {kind} {seed}", flush=True)
    x, y = _images(kind, seed, H, W)
    _, d = rga.image_loss(torch.tensor(x[None]).cuda(), torch.tensor(y[None]).cuda(), 1.0)
    got = -d[0].cpu().numpy().astype(np.float64) * (H * W)
    x64 = torch.tensor(x[None].astype(np.float64), requires_grad=True)
    loss = ref64.image_loss(x64, torch.tensor(y[None].astype(np.float64)), 1.0)
    want = -torch.autograd.grad(loss, x64)[0][0].numpy() * (H * W)
    err = np.linalg.norm(got - want)
    limit = np.linalg.norm(_gradient32(x, y) - want)
    print(f"[ssim accuracy]   {err / np.linalg.norm(want):.3e}, FP32 formula "
          f"{limit / np.linalg.norm(want):.3e}", flush=True)
    assert err <= 1.03 * limit
