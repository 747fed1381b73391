"""GPU: the coarsest solve of levels of more than 1,024 rows, for one vector, where its
kernel changes shape (16 rows a workgroup, tiles of 512 columns): z_i is the sum over
k ascending of (A^-1 e_k)_i r_k, and its time."""
import sys
import time

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import assert_same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("nu,nv", [(32, 32), (41, 25), (48, 32), (53, 29), (64, 32), (683, 3), (197, 13), (53, 47), (63, 65), (64, 64)])
def test_direct_solve(nu, nv):
    _say(f"[gpu] direct solve of {nu * nv} rows")
    from paper_2307_04886_amd.binding import default_options, from_problem
    prob = synth.small_torus(nu, nv)
    gpu, _ = from_problem(prob, default_options(min_coarse_points=prob.n))
    assert gpu.num_levels == 1
    inv = gpu.export(0, "coarse_inverse")
    R = np.random.default_rng(6).uniform(-1, 1, (2, prob.n))
    for precision, dt in (("f64", np.float64), ("f32", np.float32)):
        Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
        for q in range(2):
            r = R[q].astype(dt).astype(np.float64)
            x = np.zeros(prob.n)
            for k in range(prob.n):
                x = x + inv[k] * r[k]
            z = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
            assert_same_bits(x.astype(dt).astype(np.float64), z, f"{prob.n} rows, {precision}")
            assert_same_bits(z, Z[q], f"{prob.n} rows, {precision}, batched")


def test_direct_solve_time():
    """4,032 rows: the inverse is 130 MB, 25 us of the memory's rate, and a row's sum a
    chain of 4,032 additions, 14 us.  With two rows a workgroup, 16 of a cache line's
    128 bytes, a cycle took 385 us (and one lane a row from memory 212)."""
    from paper_2307_04886_amd.binding import default_options, from_problem
    prob = synth.small_torus(64, 63)
    gpu, _ = from_problem(prob, default_options(min_coarse_points=prob.n))
    r = torch.from_numpy(np.random.default_rng(7).uniform(-1, 1, prob.n)).cuda()
    z = torch.empty_like(r)
    for precision in ("f64", "f32"):
        gpu.precondition(r, z, precision=precision)
        best = float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                gpu.precondition(r, z, precision=precision)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 10)
        _say(f"[gpu] direct solve of 4032 rows, {precision}: {best * 1e6:.0f} us")
        assert best < 200e-6
