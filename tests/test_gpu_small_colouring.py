"""GPU: the colouring of a small level in one workgroup where its rows change
shape (entries shared by 16 lanes: rows of 1 to 64 entries and longer ones, more
than 32 and more than 64 colours), against the oracle's colours, exactly."""
import sys

import numpy as np
import pytest

import oracle
from synth.operators import Problem
from tests.test_gpu_pcg import both

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def star_of_cliques(n, clique, seed=5):
    """A path of n points whose first `clique` points are all coupled to each other."""
    rng = np.random.default_rng(seed)
    pts = np.stack([np.arange(n, dtype=float), rng.uniform(0, 0.1, n), rng.uniform(0, 0.1, n)], axis=1)
    E = {(i, i + 1) for i in range(n - 1)} | {(i, j) for i in range(clique) for j in range(i + 1, clique)}
    edges = np.array(sorted(E), dtype=np.int32)
    A = np.zeros((n, n))
    A[edges[:, 0], edges[:, 1]] = A[edges[:, 1], edges[:, 0]] = -1.0
    A[np.arange(n), np.arange(n)] = 1.0 - A.sum(axis=1)
    mask = A != 0
    indptr = np.concatenate([[0], np.cumsum(mask.sum(axis=1))]).astype(np.int32)
    r, c = np.nonzero(mask)
    return Problem("cliques", pts, edges, indptr, c.astype(np.int32), A[r, c], rng.uniform(-1, 1, n))


@pytest.mark.parametrize("n,clique", [(65, 3), (200, 17), (300, 40), (300, 63), (300, 64), (300, 70), (700, 130)])
def test_small_colouring(n, clique):
    print(f"[gpu] small colouring {n} {clique}", flush=True)
    sys.stdout.flush()
    prob = star_of_cliques(n, clique)
    orc, gpu = both(prob, min_coarse_points=10)
    assert gpu.num_levels == orc.num_levels > 1
    for l in range(gpu.num_levels - 1):
        assert np.array_equal(gpu.export(l, "colors"), orc.export(l, oracle.COLORS)), f"level {l}"
    assert gpu.sizes(0)["colors"] >= clique
