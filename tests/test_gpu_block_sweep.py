"""GPU parity of the block sweeps at the shapes where their kernel changes: row
widths of up to 58 entries (2 to 4 entries a lane, sums of 8 to 64 terms),
colours of more rows than a step takes, blocks whose matrix does not fit in LDS
(in double only, and in both precisions).  Every operation is the oracle's in its
order, so the results are compared bit for bit.
"""
import dataclasses
import sys

import numpy as np
import pytest

import oracle
import synth
from synth import configs, meshes
from tests.test_gpu_parity import assert_same_bits
from tests.test_gpu_pcg import PREC, both

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def uneven_torus(nu, nv, a):
    """A torus whose points crowd around u = pi (spacing 1 + a cos u): blocks of 1 to 366 rows."""
    pts, faces = meshes.torus_grid(nu, nv)
    u = np.arctan2(pts[:, 1], pts[:, 0])
    rho = np.hypot(pts[:, 0], pts[:, 1])
    u = u + a * np.sin(u)
    p = np.stack([rho * np.cos(u), rho * np.sin(u), pts[:, 2]], axis=1)
    return configs._mesh_problem("uneven_torus", p, faces, 1e-3, 0)


CASES = {
    "uneven": (lambda: uneven_torus(256, 200, 0.995), {}),                       # 10 to 29 entries, 366 rows
    "cloud8": (lambda: synth.small_pointcloud(45000), dict(coarsening_ratio=0.5)),          # 11 to 33 entries
    "cloud24": (lambda: synth.small_pointcloud(45000, 24), dict(coarsening_ratio=0.5)),     # 24 to 58 entries
}


@pytest.mark.parametrize("name", list(CASES))
def test_block_sweep(name):
    make, opt = CASES[name]
    prob = make()
    orc, gpu = both(prob, min_coarse_points=500, **opt)
    assert any(gpu.sizes(l)["blocks"] and gpu.sizes(l)["n"] > 4096 for l in range(gpu.num_levels))
    r = np.random.default_rng(31).uniform(-1, 1, prob.n)
    for precision in ("f64", "f32"):
        _say(f"[gpu] block sweep {name} {precision}")
        zo = orc.precondition(r, PREC[precision])
        zg = gpu.precondition(torch.from_numpy(r).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(zo, zg, f"{name} {precision}")
        Z = gpu.precondition_batched(torch.from_numpy(np.stack([r, -r, r])).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(zo, Z[2], f"{name} {precision} batched")
    _say(f"[gpu] block sweep {name} V-cycles")
    xo = orc.solve(prob.rhs, tol=0.0, max_iters=2)[0]
    xg = gpu.solve(torch.from_numpy(prob.rhs).cuda(), tol=0.0, max_iters=2)[0].cpu().numpy()
    assert_same_bits(xo, xg, name)
    # new values: the layouts' values are rebuilt
    orc2 = oracle.Hierarchy.from_problem(dataclasses.replace(prob, data=2.0 * prob.data),
                                         oracle.default_options(min_coarse_points=500, **opt))
    gpu.update_matrix(torch.from_numpy(2.0 * prob.data).cuda())
    z2 = gpu.precondition(torch.from_numpy(r).cuda()).cpu().numpy()
    assert_same_bits(orc2.precondition(r, PREC["f64"]), z2, f"{name} updated")
