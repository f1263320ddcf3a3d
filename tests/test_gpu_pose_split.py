"""The skinning matrices' gradient where its joints are split over workgroups: one joint
to 256, at the numbers of Gaussians at which the split changes, Gaussians and joints in no
order, against FP64 sums.  An entry is within 1e-5 of the sum of its absolute terms."""

import numpy as np
import pytest
import torch

from paper_2407_10707_amd import rga

pytestmark = pytest.mark.gpu


def _draw(n, J):
    rng = np.random.default_rng(n + J)
    jidx = rng.integers(-1, J + 1, (4, n)).astype(np.int32)     # with joints that do not exist
    jw = rng.random((4, n)).astype(np.float32)
    x, gx = rng.normal(size=(2, 3, n)).astype(np.float32)
    return jidx, jw, x, gx


@pytest.mark.parametrize("n,J", [(1, 1), (1, 256), (300, 5), (300, 255), (513, 9), (513, 256),
                                 (6890, 24), (20000, 30), (65000, 256), (98304, 24),
                                 (98305, 24), (196609, 24)])
def test_against_fp64(n, J):
    print(f"[pose split] {n} {J}", flush=True)
    jidx, jw, x, gx = _draw(n, J)
    got = rga.lbs_skin_pose_grad(J, *(torch.as_tensor(a).cuda() for a in (jidx, jw, x, gx)))
    w = np.zeros((J, n))
    for s in range(4):
        ok = (jidx[s] >= 0) & (jidx[s] < J)
        np.add.at(w, (jidx[s][ok], np.arange(n)[ok]), jw[s][ok].astype(np.float64))

    def terms(f):
        M = f(gx.astype(np.float64))[:, None] * np.concatenate([f(x.astype(np.float64)),
                                                                np.ones((1, n))])[None]
        return (w @ M.reshape(12, n).T).reshape(J, 3, 4)

    want, size = terms(lambda a: a), terms(np.abs)
    assert np.all(np.abs(got.cpu().numpy().reshape(J, 3, 4) - want) <= 1e-5 * size + 1e-12)


def test_few_gaussians_and_many_joints():
    """300 Gaussians, 256 joints in no order: 83 us where one workgroup walked all of a
    wave's joints, 14 with the joints split; the fastest of twenty is below 30 us."""
    a = [torch.as_tensor(v).cuda() for v in _draw(300, 256)]
    best = 1e9
    rga.timing_filter(None)
    rga.timing_enable(True)
    for _ in range(20):
        rga.timing_reset()
        rga.lbs_skin_pose_grad(256, *a)
        best = min(best, 1e3 * sum(rga.timing_read(k)[0] for k in
                                   ("lbs_pose_grad", "lbs_pose_grad_final")))
    rga.timing_enable(False)
    print(f"[pose split] {best:.1f} us", flush=True)
    assert best < 30
