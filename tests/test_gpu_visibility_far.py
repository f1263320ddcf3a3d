"""Triangles whose projected coordinates leave the 32-bit integers (view directions of
length 10^7 and 10^9; the conversion ends at the lowest and highest integer): the ring
route's test by bounding box keeps what the route in place rasterizes.  The same
triangles, without and with as many degenerate ones behind them as choose the ring
route, mark the same vertices."""

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga, synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("length", [1.0, 1e7, 1e9])
def test_rings_keep_what_lies_far_out(length):
    print(f"[vis far] {length}", flush=True)
    res, nf = 16, 200
    v, f = synth.body_mesh(7, 4)
    v, f = np.asarray(v, np.float32).T, np.asarray(f, np.int32)[::5][:nf]
    nv = v.shape[1]
    rng = np.random.default_rng(9)
    d = rng.normal(size=(24, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True) * length).astype(np.float32)
    knn = dev(np.arange(nv, dtype=np.int32)[:, None])
    more = np.concatenate([f, np.zeros((res * res + 1 - len(f), 3), np.int32)])
    assert len(f) <= res * res < len(more)
    raw = [rga.mesh_visibility(dev(v), dev(t), dev(d), res, knn, want_raw=True)[1]
           for t in (f, more)]
    assert bool((raw[0] != 0).any())
    assert torch.equal(*raw)
