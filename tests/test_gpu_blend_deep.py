"""Deep lists on a few tiles of a larger image, which are walked in parts side by
side: lists of 511 to 513 entries (one part or two), of several parts of 256, of more
than 32 parts, of more entries than 128 parts of 1,024 hold, beside tiles with short lists and empty
ones, with the tile sort in one pass and in two (more than 4,096 tiles), splats
that stop a pixel early and that never do; two blends of one binning, and a frame
whose lists do not fit the workspace.

Image and T_final against the FP32 mirror with the bounds of test_gpu_blend_lists:
1e-5 + 8 (k + 2) 2^-24 relative (k splats composited into the pixel) wherever no
decision of the pixel is within 1e-4 of its threshold.  Gradients (no upstream at
the other pixels) element by element within 1e-4 |g| + 1e-3 RMS and 1e-4 relative
L2 of those of the same lists in one walk, which takes the same FP32 decisions: a
part grows with the entries of all lists, so splats on further tiles, which the
lists of these do not meet, make every list a single part."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import cpu
from paper_2407_10707_amd import rga, synth
from tests import helpers

pytestmark = pytest.mark.gpu

# splats in the deep part and elsewhere, image, half extent of the deep part (of the
# image's height), log scale, opacities, longest list at least
CASES = [(511, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 511),
         (512, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 512),
         (513, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 513),
         (700, 500, 70, 45, 0.3, -1.5, (0.005, 0.3), 600),
         (16_500, 500, 70, 45, 0.2, -3.0, (0.004, 0.012), 16_000),
         (2047, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 2047),
         (2048, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 2048),
         (2049, 0, 16, 16, 0.4, -2.0, (0.005, 0.06), 2049),
         (2300, 200, 70, 45, 0.3, -1.5, (0.3, 0.95), 2200),
         (4500, 300, 96, 50, 0.2, -3.2, (0.005, 0.03), 3000),
         (36_000, 500, 70, 45, 0.2, -3.0, (0.004, 0.012), 35_000),
         (36_000, 500, 70, 45, 0.2, -3.0, (0.3, 0.95), 35_000),
         (140_000, 0, 20, 16, 0.3, -3.0, (0.004, 0.005), 135_000),
         (9000, 400, 1050, 1040, 0.01, -5.0, (0.01, 0.4), 8500)]
EXTRA = 256       # further tiles, each with all of the further splats: 256 x 256 pixels


def _scene(n, rest, width, height, half, scale, opac):
    rng = np.random.default_rng([43, n, rest, width])
    cam = synth.default_camera(width, height)
    deep = rng.uniform(-half, half, (2, n))
    wide = rng.uniform(-1, 1, (2, rest)) * np.array([[width / height], [1.0]])
    x = np.concatenate([np.concatenate([deep, wide], 1), rng.uniform(-0.2, 0.2, (1, n + rest))])
    n += rest
    order = rng.permutation(n)
    return cam, (np.ascontiguousarray(x[:, order], np.float32), _eye(n),
                 rng.normal(size=(4, n)).astype(np.float32),
                 rng.normal(scale, 0.2, (3, n)).astype(np.float32),
                 rng.uniform(*opac, n).astype(np.float32),
                 rng.random((3, n)).astype(np.float32), np.ones(n, np.uint8))


def _eye(n):
    return np.tile(np.eye(3, dtype=np.float32).reshape(9, 1), (1, n))


def _forward(cam, a, capacity=None):
    dev = [torch.as_tensor(v).cuda() for v in a]
    n = a[0].shape[1]
    ws = rga.SplatWorkspace(n, cam.width, cam.height, capacity or 12 * n + 1024, "cuda")
    return dev, ws, rga.splat_forward(cam, *dev, ws)


def _beside(cam, a, longest):
    """The same splats on a wider image, whose further tiles take as many entries
    as make the longest list a single part."""
    m = 128 * (longest + 64) // EXTRA + 1
    left = (cam.width + 15) // 16 * 16
    wide = dataclasses.replace(cam, width=left + 16 * (EXTRA // 16) + 16,
                               height=max(cam.height, 16 * (EXTRA // 16)))
    # at depth 3 before the camera, a disc that faces it over all of the further tiles
    R, t = np.asarray(cam.R, np.float64).reshape(3, 3), np.asarray(cam.t, np.float64)
    depth, radius = 3.0, 120.0
    c = np.array([(left + 136 - cam.cx) / cam.fx * depth, (128 - cam.cy) / cam.fy * depth, depth])
    x = np.repeat((R.T @ (c - t))[:, None], m, 1)
    sigma = radius / np.sqrt(2 * np.log(255 * 0.01)) / cam.fx * depth
    extra = (x, _eye(m), np.repeat(np.array([[1.0], [0], [0], [0]]), m, 1),
             np.repeat(np.log([[sigma], [sigma], [1e-4]]), m, 1), np.full(m, 0.01), np.full((3, m), 0.5),
             np.ones(m, np.uint8))
    both = [np.ascontiguousarray(np.concatenate([v, e.astype(v.dtype)], -1))
            for v, e in zip(a, extra)]
    return wide, both


@pytest.mark.parametrize("case", CASES)
def test_deep_lists(case):
    print(f"[blend deep] {case}", flush=True)
    cam, a = _scene(*case[:7])
    x, A, q, log_s, opac, col, front = a
    n = x.shape[1]
    dev, ws, (img, T) = _forward(cam, a)
    pre = cpu.splat_preprocess(cam, x, A, q, log_s, opac, front)
    keys, vals, ranges = cpu.splat_bin(cam, pre)
    eimg, eT, margin, napp = cpu.composite_tiles(cam, ranges, vals, pre, opac, col,
                                                 with_applied=True)
    D = ws.count()
    assert D == len(keys) <= ws.capacity
    longest = int((ranges[:, 1] - ranges[:, 0]).max())
    print(f"[blend deep]   longest list {longest} of {D}", flush=True)
    assert longest >= case[7]
    st = ws.state()
    assert np.array_equal(ws.view(st.sorted, (D,), torch.int32).cpu().numpy(), vals)
    gi, gT = img.cpu().numpy(), T.cpu().numpy()
    rel = 1e-5 + 8.0 * (napp + 2) * 2.0 ** -24
    ok = margin > np.maximum(1e-4, rel)
    assert not ((np.abs(gi - eimg) > rel[None] * np.abs(eimg) + 1e-6) & ok[None]).any()
    assert not ((np.abs(gT - eT) > rel * eT) & ok).any()

    wide, both = _beside(cam, a, longest)
    m = both[0].shape[1] - n
    dev1, ws1, (img1, _) = _forward(wide, both, capacity=D + 300 * m + 1024)
    D1 = ws1.count()
    assert 128 * (longest + 64) <= D1 - D <= 300 * m
    rng = np.random.default_rng(5)
    w = torch.as_tensor((rng.uniform(0.5, 1.5, eimg.shape) * ok[None]).astype(np.float32)).cuda()
    up = torch.zeros_like(img1)
    up[:, :cam.height, :cam.width] = w
    ref = rga.splat_backward(wide, *dev1, ws1, img1, up, want_dA=True)
    for _ in range(2):          # the second backward finds the sums as the first did
        g = rga.splat_backward(cam, *dev, ws, img, w, want_dA=True)
        for k, v in g.items():
            helpers.check_grad(k, v.cpu().numpy(), ref[k][..., :n].cpu().numpy())


def test_two_blends_of_one_binning():
    print("[blend deep] two blends", flush=True)
    cam, a = _scene(4500, 300, 96, 50, 0.2, -3.2, (0.005, 0.3))
    dev, ws, first = _forward(cam, a)
    other = torch.rand(dev[5].shape, device="cuda")
    for col in (other, dev[5], other):
        img, T = rga.splat_blend(cam, col, ws)
        b = [v.cpu().numpy() if torch.is_tensor(v) else v for v in dev]
        b[5] = col.cpu().numpy()
        _, _, (want, wT) = _forward(cam, b)
        assert torch.equal(img, want) and torch.equal(T, wT)


def test_deep_lists_that_do_not_fit():
    print("[blend deep] overflow", flush=True)
    cam, a = _scene(4500, 300, 96, 50, 0.2, -3.2, (0.005, 0.3))
    dev, ws, (img, T) = _forward(cam, a, capacity=5000)
    assert ws.count() > 5000
    assert bool(img.isnan().all()) and bool(T.isnan().all())
    g = rga.splat_backward(cam, *dev, ws, img, torch.ones_like(img))
    assert all(bool(v.isnan().all()) for v in g.values() if v is not None)


def test_a_deep_list_is_shared_out():
    """The lists of a few tiles of a 600 x 600 image, 50,000 entries and more, whose
    pixels do not stop: one walk takes over 1 ms, the parts 0.1 ms; the fastest of ten
    blends and of ten adjoints is below 0.5 ms."""
    print("[blend deep] time", flush=True)
    cam, a = _scene(100_000, 0, 600, 600, 0.01, -5.5, (0.004, 0.005))
    dev, ws, (img, _) = _forward(cam, a)
    st = ws.state()
    r = ws.view(st.ranges, (38 * 38, 2), torch.int32)
    assert int((r[:, 1] - r[:, 0]).max()) > 50_000
    up = torch.ones_like(img)
    best = dict(blend=1e9, blend_bwd=1e9)
    rga.timing_filter(None)
    rga.timing_enable(True)
    for _ in range(10):
        rga.timing_reset()
        rga.splat_blend(cam, dev[5], ws)
        rga.splat_backward(cam, *dev, ws, img, up)
        for k in best:
            best[k] = min(best[k], rga.timing_read(k)[0])
    rga.timing_enable(False)
    print(f"[blend deep]   {best}", flush=True)
    assert max(best.values()) < 0.5
