"""Visibility of meshes at the edges of the raster's two routes (triangles in
place; triangles gathered in rings, with and without the table of projected
vertices), of its batches of 8192 triangles, and of the filters' one and four
words per thread.  Bits and counts are equal to the CPU oracle's."""

import numpy as np
import pytest
import torch

from oracle import cpu
from paper_2407_10707_amd import rga, synth

pytestmark = pytest.mark.gpu

# (segments, rings, triangles kept, views, res, numbering of a body mesh or size of a random one)
CASES = [
    (7, 4, 512, 40, 16, "body"),        # 2 res^2 triangles: in place
    (7, 4, 513, 40, 16, "body"),        # one more: rings
    (7, 4, 1008, 33, 1, "body"),        # one pixel
    (18, 21, 8192, 24, 32, "body"),     # one whole batch
    (18, 21, 8193, 24, 32, "body"),     # one triangle in the second
    (18, 21, 13608, 24, 64, "shuffled"),     # all vertices in the table
    (48, 46, 79488, 6, 128, "shuffled"),     # ranges longer than the table
    (48, 46, 79488, 6, 128, "body"),
    (48, 46, 79488, 230, 64, "body"),   # four words per thread, ragged views
    (0, 0, 40000, 5, 128, 216000),      # no room for a table
    (0, 0, 40000, 5, 128, 250000),      # nor for rings
]


@pytest.mark.parametrize("case", CASES)
def test_visibility_bit_exact(case):
    print(f"[vis meshes] {case}", flush=True)
    seg, rings, nf, V, res, numbering = case
    rng = np.random.default_rng(7)
    if seg:
        v, f = synth.body_mesh(seg, rings)
        v = np.asarray(v, np.float32)
        v = v if v.shape[0] == 3 else v.T
        f = np.asarray(f, np.int32)
        nv = v.shape[1]
        knn = np.clip(np.arange(nv)[:, None] + np.arange(-9, 10)[None], 0, nv - 1)
    else:
        nv = numbering
        v = rng.normal(size=(3, nv)).astype(np.float32)
        f = (rng.integers(0, nv - 3, size=nf)[:, None] + np.arange(3)[None]).astype(np.int32)
        knn = np.arange(nv)[:, None]
    if numbering == "shuffled":
        perm = rng.permutation(nv)
        back = np.argsort(perm)
        v, f, knn = v[:, perm], back[f], back[knn[perm]]
    assert nf <= len(f)
    f = np.ascontiguousarray(f[:nf], np.int32)
    v, knn = np.ascontiguousarray(v), np.ascontiguousarray(knn, np.int32)
    d = rng.normal(size=(V, 3)).astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    dev = lambda a: torch.from_numpy(a).cuda()
    count, raw = rga.mesh_visibility(dev(v), dev(f), dev(d), res, dev(knn), want_raw=True)
    eraw, ecnt = cpu.mesh_visibility(v, f, d, res, knn)
    assert np.array_equal(raw.cpu().numpy().view(np.uint32), eraw)
    assert np.array_equal(count.cpu().numpy(), ecnt)
