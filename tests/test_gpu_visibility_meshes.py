"""Visibility of meshes at the edges of the raster's two routes (triangles in
place; triangles gathered in rings, with and without the table of the vertices'
places), of its batches of 16384 triangles, of the views per workgroup and of the
filters' one and four words per thread; with frames and directions that take no
table, and in a workspace without room for the raster's copies.  Bits and counts
are equal to the CPU oracle's."""

import numpy as np
import pytest
import torch

from oracle import cpu
from paper_2407_10707_amd import rga, synth

pytestmark = pytest.mark.gpu

# (segments, rings, triangles kept, views, res, numbering of a body mesh or size of a random one)
CASES = [
    (7, 4, 256, 40, 16, "body"),        # res^2 triangles: in place
    (7, 4, 257, 40, 16, "body"),        # one more: rings
    (7, 4, 512, 40, 16, "body"),
    (7, 4, 1008, 33, 1, "body"),        # one pixel
    (7, 4, 200, 261, 16, "body"),       # more views than compute units, in place
    (7, 4, 900, 517, 16, "body"),       # three views in a workgroup, rings
    (18, 21, 8193, 24, 32, "body"),
    (18, 21, 13608, 24, 64, "shuffled"),     # all vertices in the table
    (48, 46, 16384, 6, 96, "body"),     # one whole batch
    (48, 46, 16385, 6, 96, "body"),     # one triangle in the second
    (48, 46, 79488, 6, 128, "shuffled"),     # ranges longer than the table
    (48, 46, 79488, 6, 128, "body"),
    (48, 46, 79488, 300, 64, "body"),   # four words per thread, ragged views
    (0, 0, 40000, 5, 128, 216000),      # no room for a table
    (0, 0, 40000, 5, 128, 250000),      # nor for rings
]


def _mesh(seg, rings, nf, V, numbering):
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
    d = rng.normal(size=(V, 3)).astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return (np.ascontiguousarray(v), np.ascontiguousarray(f[:nf], np.int32), d,
            np.ascontiguousarray(knn, np.int32))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _equal(count, raw, v, f, d, res, knn):
    eraw, ecnt = cpu.mesh_visibility(v, f, d, res, knn)
    assert np.array_equal(raw.cpu().numpy().view(np.uint32), eraw)
    assert np.array_equal(count.cpu().numpy(), ecnt)


@pytest.mark.parametrize("case", CASES)
def test_visibility_bit_exact(case):
    print(f"[vis meshes] {case}", flush=True)
    seg, rings, nf, V, res, numbering = case
    v, f, d, knn = _mesh(seg, rings, nf, V, numbering)
    count, raw = rga.mesh_visibility(dev(v), dev(f), dev(d), res, dev(knn), want_raw=True)
    _equal(count, raw, v, f, d, res, knn)


# scale of the mesh, of the view directions: the frame's radius from squares below
# the normal floats (and 0, and above them all); directions that are no unit vectors
@pytest.mark.parametrize("scale,length", [(3e-23, 1), (1e-20, 1), (1e-30, 1), (3e19, 1),
                                          (1, 1.5), (1, 0.3), (1, 1.001)])
def test_visibility_without_a_frame(scale, length):
    print(f"[vis meshes] scale {scale} length {length}", flush=True)
    v, f, d, knn = _mesh(18, 21, 13608, 9, "body")
    v, d = (v * np.float32(scale)).astype(np.float32), (d * np.float32(length)).astype(np.float32)
    count, raw = rga.mesh_visibility(dev(v), dev(f), dev(d), 64, dev(knn), want_raw=True)
    _equal(count, raw, v, f, d, 64, knn)


# views, bytes less than the workspace function gives
@pytest.mark.parametrize("V,less", [(9, 0), (9, 15), (300, 0)])
def test_visibility_small_workspace(V, less):
    print(f"[vis meshes] workspace {V} {less}", flush=True)
    v, f, d, knn = _mesh(18, 21, 13608, V, "body")
    nv, words = v.shape[1], (V + 31) // 32
    up = lambda b: (b + 255) // 256 * 256
    layout = 256 + up(V * ((nv + 31) // 32) * 4) + 3 * up(nv * words * 4)
    full = int(rga.lib().mesh_visibility_workspace(nv, V))
    assert full >= layout
    size = layout if less == 0 else full - less
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    count = torch.empty((nv, V), dtype=torch.uint8, device="cuda")
    raw = torch.empty((nv, words), dtype=torch.int32, device="cuda")
    a = [dev(v), dev(f), dev(d), dev(knn)]
    st = torch.cuda.current_stream().cuda_stream
    call = lambda n: rga.lib().mesh_visibility(
        st, nv, len(f), a[0].data_ptr(), a[1].data_ptr(), V, a[2].data_ptr(), 64, a[3].data_ptr(),
        knn.shape[1], raw.data_ptr(), count.data_ptr(), ws.data_ptr(), n)
    assert call(size) == 0
    _equal(count, raw, v, f, d, 64, knn)
    assert call(layout - 1) == -2


# several views in a workgroup, whose z-buffer the depth test leaves as it is
@pytest.mark.parametrize("nf", [200, 900])
def test_shadow_maps_share_workgroups(nf):
    print(f"[vis meshes] shadow {nf}", flush=True)
    v, f, d, knn = _mesh(7, 4, nf, 517, "body")
    count, raw = rga.mesh_visibility(dev(v), dev(f), dev(d), 16, dev(knn), want_raw=True,
                                     shadow_bias_px=1.5)
    eraw, ecnt = cpu.mesh_visibility_shadow(v, f, d, 16, knn, 1.5)
    assert np.array_equal(raw.cpu().numpy().view(np.uint32), eraw)
    assert np.array_equal(count.cpu().numpy(), ecnt)
