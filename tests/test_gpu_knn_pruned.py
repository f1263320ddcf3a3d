"""The search for at most four neighbours where its pruning of rows and cells can
go wrong: points in a few crowded cells, on lattices (ties, and queries on cell
boundaries), on a line and in a plane, queries far outside and in empty cells,
ragged query counts, and queries in the order of their cells and in none.
Neighbours and their order are the oracle's bit for bit (FP32 distances, ties by
index); weights within 2e-6 relative of the FP64 weights of those distances."""

import numpy as np
import pytest

from tests.test_gpu_knn import _check

pytestmark = pytest.mark.gpu


def _points(kind, rng):
    if kind == "crowded":
        c = rng.random((3, 12)).astype(np.float32)
        r = c[:, rng.integers(0, 12, 3000)] + rng.normal(size=(3, 3000)) * 0.01
    elif kind == "lattice":
        g = np.arange(12) * 0.25
        r = np.stack(np.meshgrid(g, g, g, indexing="ij")).reshape(3, -1)
    elif kind == "line":
        r = np.stack([rng.random(2000) * 100, np.zeros(2000), np.ones(2000)])
    elif kind == "plane":
        r = np.stack([rng.random(5000), rng.random(5000), np.full(5000, 0.5)])
    else:
        r = rng.random((3, 20000)) * np.array([[1.0], [3.0], [0.3]]) - 1.0
    return r.astype(np.float32)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", ["crowded", "lattice", "line", "plane", "box"])
def test_pruned_search(kind, k):
    rng = np.random.default_rng(17 * k + len(kind))
    r = _points(kind, rng)
    lo, hi = r.min(1, keepdims=True), r.max(1, keepdims=True)
    near = r[:, rng.integers(0, r.shape[1], 701)] + rng.normal(size=(3, 701)) * 0.02
    inside = lo + (hi - lo) * rng.random((3, 400))
    grid = np.round(8 * (lo + (hi - lo) * rng.random((3, 300)))) / 8
    around = lo + (hi - lo) * (rng.random((3, 200)) * 3 - 1)
    far = rng.normal(size=(3, 99)) * 1e4
    q = np.concatenate([near, inside, grid, around, far, r[:, :65]], 1).astype(np.float32)
    _check(q, r, k)
    _check(np.ascontiguousarray(q[:, np.lexsort(q)]), r, k)
    for n in (1, 15, 17):
        _check(np.ascontiguousarray(q[:, :n]), r, k)
