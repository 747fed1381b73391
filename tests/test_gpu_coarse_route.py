"""GPU: where the batched cycle restricts into the coarsest level in its solve (up to
512 coarsest rows, and a vector's residual within 72 KiB) and where it does not: the
route taken, and the single-vector cycle's bits on both."""
import sys

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import assert_same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {                                    # mesh, options, fused in float, in double
    "small": (lambda: synth.small_torus(42, 42), {}, True, True),
    "torus60": (lambda: synth.small_torus(60, 60), {"min_coarse_points": 500}, True, True),
    "torus64": (lambda: synth.small_torus(64, 64), {}, False, False),                  # 549 rows
    "staged_f32": (lambda: synth.small_pointcloud(11000, 24), {}, True, False),
    "unstaged": (lambda: synth.small_pointcloud(19000, 44), {}, False, False),
    "one_level": (lambda: synth.small_torus(20, 20), {}, False, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_coarse_route(name):
    print(f"[gpu] coarse route {name}", flush=True)
    sys.stdout.flush()
    from paper_2307_04886_amd.binding import default_options, from_problem
    make, opt, f32, f64 = CASES[name]
    prob = make()
    gpu, _ = from_problem(prob, default_options(**opt))
    nl = gpu.num_levels
    nc, nf = gpu.sizes(nl - 1)["n"], gpu.sizes(max(nl - 2, 0))["n"]
    assert (nl > 1 and nc <= 512 and 4 * nf <= 72 * 1024) == f32
    assert (nl > 1 and nc <= 512 and 8 * nf <= 72 * 1024) == f64
    for l in range(nl):
        last = l + 2 == nl
        assert gpu.routes(l)["coarse_fused_f32"] == (last and f32)
        assert gpu.routes(l)["coarse_fused_f64"] == (last and f64)
    R = np.random.default_rng(11).uniform(-1, 1, (9, prob.n))
    for precision in ("f64", "f32"):
        Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
        for q in (0, 5, 8):
            z = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
            assert_same_bits(z, Z[q], f"{name} {precision} {q}")
