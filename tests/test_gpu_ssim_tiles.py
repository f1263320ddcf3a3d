"""The image loss at the edges of its 32 x 54 pixel tiles and of their division
over the XCDs (fewer tiles than eight, eight, one more, a remainder), with and
without the gradient, against the FP64 oracle.  Tolerances as derived in
test_gpu_ssim for images with texture: the loss within 2e-6, the gradient within
2e-5 of its largest value."""

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga
from tests.test_gpu_ssim import _check

pytestmark = pytest.mark.gpu

# channels, height, width
SHAPES = [(1, 54, 32), (1, 55, 33), (3, 53, 31), (1, 108, 128), (2, 109, 65), (3, 5, 300),
          (3, 300, 5), (9, 60, 20), (1, 49, 37), (1, 59, 42)]


@pytest.mark.parametrize("shape", SHAPES)
def test_tile_edges(shape):
    rng = np.random.default_rng(sum(shape))
    x, y = rng.uniform(0, 1, shape), rng.uniform(0, 1, shape)
    _check(x, y, 0.2, 2e-5)
    xt = torch.tensor(x, dtype=torch.float32).cuda()
    yt = torch.tensor(y, dtype=torch.float32).cuda()
    alone, none = rga.image_loss(xt, yt, 0.2, want_grad=False)
    both, _ = rga.image_loss(xt, yt, 0.2)
    assert none is None and torch.equal(alone, both)
