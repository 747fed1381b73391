"""GPU: meshes whose points come in an order without locality (the finest rows are
then numbered by coarse cell within a colour) against the oracle, and against the
same mesh in grid order (numbered by index): cycles bit for bit, CG by its
iteration count."""
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import synth
from synth.operators import Problem
from tests.test_gpu_parity import assert_same_bits
from tests.test_gpu_pcg import PREC, both, compare_pcg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def reordered(prob, order):
    """Point i of the result is point order[i] of prob."""
    inv = np.empty(prob.n, dtype=np.int64)
    inv[order] = np.arange(prob.n)
    e = np.sort(inv[prob.edges], axis=1)
    e = e[np.lexsort((e[:, 1], e[:, 0]))].astype(np.int32)
    A = sp.csr_matrix((prob.data, prob.indices, prob.indptr), shape=(prob.n, prob.n))[order][:, order].tocsr()
    A.sort_indices()
    return Problem(prob.name + "_reordered", np.ascontiguousarray(prob.points[order]), e, A.indptr.astype(np.int32),
                   A.indices.astype(np.int32), A.data, prob.rhs[order].copy())


@pytest.mark.parametrize("kind", ["grid", "random", "strided", "halves"])
def test_point_order(kind):
    prob = synth.small_torus(256, 160)
    n = prob.n
    rng = np.random.default_rng(3)
    order = {"grid": np.arange(n), "random": rng.permutation(n),
             "strided": np.argsort(np.arange(n) * 7919 % n, kind="stable"),
             "halves": np.concatenate([np.arange(n // 2), n // 2 + rng.permutation(n - n // 2)])}[kind]
    prob = reordered(prob, order)
    orc, gpu = both(prob, min_coarse_points=300)
    assert gpu.sizes(1)["blocks"]
    r = rng.uniform(-1, 1, n)
    for precision in ("f64", "f32"):
        print(f"[gpu] point order {kind} {precision}", flush=True)
        sys.stdout.flush()
        zo = orc.precondition(r, PREC[precision])
        zg = gpu.precondition(torch.from_numpy(r).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(zo, zg, f"{kind} {precision}")
        Z = gpu.precondition_batched(torch.from_numpy(np.stack([r, r])).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(zo, Z[1], f"{kind} {precision} batched")
        compare_pcg(orc, gpu, prob, precision)
    xo = orc.solve(prob.rhs, tol=0.0, max_iters=2)[0]
    xg = gpu.solve(torch.from_numpy(prob.rhs).cuda(), tol=0.0, max_iters=2)[0].cpu().numpy()
    assert_same_bits(xo, xg, kind)
    orc2 = oracle.Hierarchy.from_problem(Problem(prob.name, prob.points, prob.edges, prob.indptr, prob.indices,
                                                 3.0 * prob.data, prob.rhs), oracle.default_options(min_coarse_points=300))
    gpu.update_matrix(torch.from_numpy(3.0 * prob.data).cuda())
    z2 = gpu.precondition(torch.from_numpy(r).cuda()).cpu().numpy()
    assert_same_bits(orc2.precondition(r, PREC["f64"]), z2, f"{kind} updated")
