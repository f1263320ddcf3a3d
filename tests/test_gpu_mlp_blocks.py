"""The displacement network at the edges of its blocks of 32 vertices, its
workgroups of two and the layers' chunks (as many as 256-vertex pieces, each
layer's own largest number at 39 to 40 and past 58 of them), forward and adjoint,
with the bounds and the exempt vertices of test_gpu_mlp."""

import pytest

from tests.test_gpu_mlp import _backward_check, _forward_check, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv", [32, 33, 64, 65, 96, 9985, 10240, 15000])
def test_blocks_and_chunks(nv):
    x, inp = _inputs(nv, nv)
    _forward_check(x, inp)
    _backward_check(x, inp, nv)
