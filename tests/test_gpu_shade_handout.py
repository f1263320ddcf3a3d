"""Shading where its workgroups hand their Gaussians out differently: grids of
whole groups of 8 workgroups and others, eight and sixteen waves (4096
Gaussians on 256 CUs and one more), lists filled in more than one round, the
largest direction tables, with and without a tape.

The Gaussians of a scene of 500 are repeated: each copy's colour and gradients
are bit for bit those of the 500 (one Gaussian's sums are its own wave's), which
the other tests compare with the oracle.  Where every Gaussian is there equally
often the environment gradient is that many times the scene's.  Its terms are of
one sign (albedo, tint, radiance and upstream gradient are positive), so an FP32
sum of m of them is within m 2^-24 of itself, m at most 1200 / 2 per workgroup
and entry, and the partials are added in 64 chains: 2e-4 covers both sides."""

import numpy as np
import pytest
import torch

from oracle import cpu
from paper_2407_10707_amd import rga, synth
from tests import helpers

pytestmark = pytest.mark.gpu

BASE = 500
# (n, he, we, hv, wv)
CASES = [(1, 8, 16, 4, 8), (57, 8, 16, 4, 8), (4096, 8, 16, 4, 8), (4097, 8, 16, 4, 8),
         (4100, 16, 32, 16, 32), (4500, 32, 64, 32, 32), (5000, 24, 64, 24, 64),
         (45000, 56, 62, 8, 2), (140000, 4, 8, 4, 8), (600000, 4, 8, 4, 4)]


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("case", CASES)
def test_repeated_gaussians(case):
    print(f"[shade handout] {case}", flush=True)
    n, he, we, hv, wv = case
    s = synth.micro_scene(31, BASE, 40, 48, he=he, we=we, hv=hv, wv=wv)
    xo, no, _ = cpu.lbs_f32(s["skin"], s["jidx"], s["jw"], s["pos"], s["nrm"])
    _, _, cnt = helpers.oracle_visibility(s)
    campos = s["cam"].centre.astype(np.float32)
    rng = np.random.default_rng(3)
    w = rng.uniform(0.5, 1.0, (3, BASE)).astype(np.float32)
    x0 = rng.uniform(-1.0, 1.0, (3, BASE)).astype(np.float32)
    per = [xo, no, s["albedo"], s["rough"], s["tint"], s["vidx"], s["vw"]]
    rest = (dev(cnt), s["kv"], he, we, hv, wv, dev(s["env"]), campos)
    pick = np.arange(n) % BASE

    def run(idx, taped):
        a = [dev(np.asarray(p)[..., idx]) for p in per]
        tape = rga.shade_tape(len(idx), he, we, "cuda") if taped else None
        color, front = rga.shade_gaussians(*a, *rest, tape=tape)
        g = rga.shade_gaussians_backward(*a, *rest, color, front, dev(w[:, idx]),
                                         dx_accum=dev(x0[:, idx]), tape=tape)
        torch.cuda.synchronize()
        return dict(g, color=color, front=front)

    back = torch.as_tensor(pick).cuda()
    for taped in (True, False):
        if taped and 8 * n * he * we > 4e9:
            continue
        one, many = run(np.arange(BASE), taped), run(pick, taped)
        for k in ("color", "front", "dx", "dn", "dalbedo", "drough", "dtint"):
            assert torch.equal(many[k], one[k][..., back]), (k, taped)
        if n % BASE == 0:
            want = one["denv"].double() * (n // BASE)
            assert torch.allclose(many["denv"].double(), want, rtol=2e-4, atol=0.0)
        else:
            assert bool(torch.isfinite(many["denv"]).all())


# the forward that leaves room beside it: the same colours, flags and tape
@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("case", [(4097, 8, 16, 4, 8), (20000, 8, 16, 8, 16), (33000, 8, 16, 8, 16),
                                  (9000, 16, 32, 16, 32)])
def test_beside(case, precision):
    print(f"[shade handout] beside {case} {precision}", flush=True)
    n, he, we, hv, wv = case
    s = synth.micro_scene(31, BASE, 40, 48, he=he, we=we, hv=hv, wv=wv)
    xo, no, _ = cpu.lbs_f32(s["skin"], s["jidx"], s["jw"], s["pos"], s["nrm"])
    _, _, cnt = helpers.oracle_visibility(s)
    pick = np.arange(n) % BASE
    a = [dev(np.asarray(p)[..., pick]) for p in (xo, no, s["albedo"], s["rough"], s["tint"],
                                                 s["vidx"], s["vw"])]
    rest = (dev(cnt), s["kv"], he, we, hv, wv, dev(s["env"]), s["cam"].centre.astype(np.float32))
    out = []
    for beside in (False, True):
        tape = rga.shade_tape(n, he, we, "cuda")
        tape.zero_()
        out.append((*rga.shade_gaussians(*a, *rest, precision=precision, tape=tape, beside=beside),
                    tape))
    for one, other in zip(*out):
        assert torch.equal(one, other)
