"""GPU parity of the levels swept by one workgroup and of the coarsest solve, at
the sizes where their kernels change shape: chunks of 64 rows, row widths of 8,
16 and 32 entries and longer rows, resident and streamed levels, the rows a
workgroup of the coarsest solve takes, the restriction fused or apart, its
residual staged in LDS or not.  Every operation is the oracle's in its order, so
the results are compared bit for bit.
"""
import sys

import numpy as np
import pytest

import synth
from tests.conftest import problem
from tests.test_gpu_parity import assert_same_bits
from tests.test_gpu_pcg import PREC, both

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


MAKERS = {
    "torus8x8": lambda: synth.small_torus(8, 8),           # one chunk per colour
    "torus13x5": lambda: synth.small_torus(13, 5),         # 65 rows
    "torus64x56": lambda: synth.small_torus(64, 56),       # 3584 rows
    "torus64x64": lambda: synth.small_torus(64, 64),       # the largest one-workgroup level
    "torus17x241": lambda: synth.small_torus(17, 241),     # 4097: one row too many
    "cloud1000": lambda: synth.small_pointcloud(1000),
    "cloud3500": lambda: synth.small_pointcloud(3500),     # rows of up to 16 or 32 entries
    "torus100x92": lambda: synth.small_torus(100, 92),
    "hubs64": lambda: synth.small_hubs(64, 60),            # rows longer than the buffers
}
CASES = [("torus8x8", dict(min_coarse_points=10)), ("torus13x5", dict(min_coarse_points=10, nu_pre=1, nu_post=3)),
         ("torus64x56", dict(min_coarse_points=200)), ("torus64x64", {}), ("torus64x64", dict(nu_pre=0)),
         ("torus17x241", dict(min_coarse_points=100)), ("cloud1000", dict(min_coarse_points=30)),
         ("cloud3500", dict(min_coarse_points=200)), ("hubs64", dict(min_coarse_points=300)),
         ("torus100x92", dict(min_coarse_points=1100)),                       # restriction apart: 1,2xx coarsest rows
         ("torus100x92", dict(coarsening_ratio=0.05, min_coarse_points=1000))]  # residual not staged in double


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("name,opt", CASES)
def test_small_level_cycle(name, opt, precision):
    _say(f"[gpu] small levels {name} {opt} {precision}")
    prob = MAKERS[name]()
    orc, gpu = both(prob, **opt)
    R = np.random.default_rng(5).uniform(-1, 1, (3, prob.n))
    Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
    for q in range(3):
        zo = orc.precondition(R[q], PREC[precision])
        zg = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
        assert_same_bits(zo, zg, f"{name} {precision}")
        assert_same_bits(zo, Z[q], f"{name} {precision} batched")


@pytest.mark.parametrize("name,opt", CASES)
def test_small_level_vcycles(name, opt):
    _say(f"[gpu] small levels, plain cycle {name} {opt}")
    prob = MAKERS[name]()
    orc, gpu = both(prob, **opt)
    xo = orc.solve(prob.rhs, tol=0.0, max_iters=3)[0]
    xg = gpu.solve(torch.from_numpy(prob.rhs).cuda(), tol=0.0, max_iters=3)[0].cpu().numpy()
    assert_same_bits(xo, xg, name)


@pytest.mark.parametrize("nu,nv", [(3, 3), (16, 4), (27, 19), (32, 32), (41, 25), (46, 45)])
def test_direct_solve_sizes(nu, nv):
    """One level only: z_i is the sum over k ascending of (A^-1 e_k)_i r_k."""
    _say(f"[gpu] direct solve of {nu * nv} rows")
    from paper_2307_04886_amd.binding import default_options, from_problem
    prob = synth.small_torus(nu, nv)
    gpu, _ = from_problem(prob, default_options(min_coarse_points=prob.n))
    assert gpu.num_levels == 1
    inv = gpu.export(0, "coarse_inverse")
    R = np.random.default_rng(6).uniform(-1, 1, (9, prob.n))
    for precision, dt in (("f64", np.float64), ("f32", np.float32)):
        Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
        for q in range(9):
            r = R[q].astype(dt).astype(np.float64)
            x = np.zeros(prob.n)
            for k in range(prob.n):
                x = x + inv[k] * r[k]
            assert_same_bits(x.astype(dt).astype(np.float64), Z[q], f"{prob.n} rows, {precision}, vector {q}")
