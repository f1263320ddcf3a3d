"""A camera reaches the library alike from numpy arrays of any layout, torch
tensors and nested lists; what is no device tensor is refused by name."""

import types

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga


@pytest.mark.parametrize("kind", ["f64", "f32", "transposed", "torch", "list"])
def test_camera(kind):
    R = np.arange(9, dtype=np.float64).reshape(3, 3) / 8
    t = np.array([0.5, -0.25, 3.0])
    make = dict(f64=lambda a: a, f32=lambda a: a.astype(np.float32),
                transposed=lambda a: np.asfortranarray(a), torch=torch.as_tensor,
                list=lambda a: a.tolist())[kind]
    c = rga.camera(types.SimpleNamespace(R=make(R), t=make(t), fx=2, fy=3.0, cx=1.5, cy=np.float32(2.5),
                                         width=np.int64(4), height=5))
    assert list(c.R) == R.reshape(-1).tolist() and list(c.t) == t.tolist()
    assert (c.fx, c.fy, c.cx, c.cy, c.width, c.height) == (2.0, 3.0, 1.5, 2.5, 4, 5)


@pytest.mark.parametrize("bad", [None, [1.0], np.zeros(3, np.float32), torch.zeros(3)])
def test_host_arguments_are_refused(bad):
    with pytest.raises(rga.RgaError, match="weights must be a CUDA"):
        rga._f32(bad, "weights", (3,))
