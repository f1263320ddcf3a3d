"""The image loss over more tiles than one dimension of a grid holds threads for
(2^24 tiles of 256 threads; 65,535 one-row images of 8,193 pixels have 16.8 million):
the gradient of a few channels equals that of those channels alone, which has the
same arithmetic and a divisor of its own (two roundings of 2^-24, limit 1e-6), and the
loss the mean over four shares of the channels, within 2e-6 as in test_gpu_ssim."""

import pytest
import torch

from paper_2407_10707_amd import rga

pytestmark = pytest.mark.gpu


def test_more_than_2_to_24_tiles():
    C, W = 65535, 8193
    print(f"[ssim tiles] {C} x {W}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.rand((C, 1, W), generator=g, device="cuda")
    y = torch.rand((C, 1, W), generator=g, device="cuda")
    loss, d = rga.image_loss(x, y, 0.2)
    torch.cuda.synchronize()
    shares = torch.arange(C, device="cuda").chunk(4)
    want = sum(float(rga.image_loss(x[s[0]:s[-1] + 1], y[s[0]:s[-1] + 1], 0.2,
                                    want_grad=False)[0]) * len(s) for s in shares) / C
    assert abs(float(loss) - want) <= 2e-6
    for c in (0, 1, 40000, C - 1):
        alone = rga.image_loss(x[c:c + 1], y[c:c + 1], 0.2)[1] / C
        assert bool(((d[c:c + 1] - alone).abs() <= 1e-6 * alone.abs() + 1e-6 / (C * W)).all())
    assert bool((d.abs().amax(dim=2) > 0).all())
