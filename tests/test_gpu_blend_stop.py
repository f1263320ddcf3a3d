"""The adjoint of the compositing stops where the forward stopped, also where T
passes 1e-4 within the rounding of its product: splats whose means lie exactly on a
pixel's centre (alpha is their opacity, bit for bit), with opacities chosen so that
the products of the forward (four entries at a time) and of a walk entry by entry
lie on either side of 1e-4.  With dL/dimage = 1 at that pixel alone, a splat's
dL/dcolour is its weight alpha T, and the weights of the entries that counted add up
to 1 - T_final.  An entry more or less is a weight of 1e-4 to 2e-4; the sum of up to
50 FP32 weights is within 50 x 2^-24 = 3e-6."""

import dataclasses

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga, synth

pytestmark = pytest.mark.gpu

F = np.float32
STOP = F(1e-4)


def _by_fours(o):
    """T after each entry, as the forward multiplies."""
    T, out = F(1), []
    for i in range(0, len(o), 4):
        m = [F(1) - v for v in o[i:i + 4]] + [F(1)] * (4 - len(o[i:i + 4]))
        p = [m[0], m[1] * m[0], (m[2] * m[1]) * m[0], (m[3] * m[2]) * (m[1] * m[0])]
        out += [T * v for v in p]
        T = T * p[3]
    return out[:len(o)]


def _one_by_one(o):
    T, out = F(1), []
    for v in o:
        T = T * (F(1) - v)
        out.append(T)
    return out


def _opacities(seed, above):
    """Opacities whose last entry but two passes 1e-4 in one of the products only."""
    rng = np.random.default_rng([17, seed, above])
    while True:
        n = int(rng.integers(9, 45))
        o = rng.uniform(0.02, 8.2 / n, n).astype(F)
        t = _one_by_one(o)[-1]
        if not 1.5e-4 < t < 3e-4:
            continue
        o = np.append(o, F(0))
        for _ in range(64):
            o[-1] = F(1 - 1e-4 / float(t)) + F(rng.integers(-6, 7) * 6e-8)
            a, b = _by_fours(o)[-1] >= STOP, _one_by_one(o)[-1] >= STOP
            if a != b and a == above and min(_by_fours(o)[:-1]) >= STOP:
                return np.append(o, rng.uniform(0.3, 0.5, 2)).astype(F)


@pytest.mark.parametrize("above", [True, False])
@pytest.mark.parametrize("seed", range(6))
def test_adjoint_stops_with_the_forward(seed, above):
    o = _opacities(seed, above)
    n = len(o)
    print(f"[blend stop] {seed} {above} {n}", flush=True)
    cam = dataclasses.replace(synth.default_camera(32, 32), cx=12.5, cy=9.5)
    R, t = np.asarray(cam.R, np.float64).reshape(3, 3), np.asarray(cam.t, np.float64)
    z = 2.0 + 0.01 * np.arange(n)
    x = (R.T @ (np.stack([0 * z, 0 * z, z]) - t[:, None])).astype(F)
    rng = np.random.default_rng(3)
    q = np.zeros((4, n), F)
    q[0] = 1
    dev = [torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in (
        x, np.tile(np.eye(3, dtype=F).reshape(9, 1), (1, n)), q, np.full((3, n), -3.0, F), o,
        rng.random((3, n)).astype(F), np.ones(n, np.uint8))]
    ws = rga.SplatWorkspace(n, 32, 32, 4096, "cuda")
    img, T = rga.splat_forward(cam, *dev, ws)
    st = ws.state()
    mean = ws.view(st.mean2d, (2, n), torch.float32).cpu().numpy()
    assert np.all(mean[0] == 12.5) and np.all(mean[1] == 9.5)
    got = float(T[9, 12].cpu())
    by_fours = [v for v in _by_fours(o) if v >= STOP]
    assert got == by_fours[-1]
    up = torch.zeros_like(img)
    up[0, 9, 12] = 1
    g = rga.splat_backward(cam, *dev, ws, img, up)
    w = g["dcolor"][0].cpu().numpy().astype(np.float64)
    print(f"[blend stop]   T {got:.9e} weights {w.sum():.9e}", flush=True)
    assert np.count_nonzero(w) == len(by_fours)
    assert abs(w.sum() - (1.0 - got)) < 3e-6
