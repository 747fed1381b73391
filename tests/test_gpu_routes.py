"""GPU: the forms of the cycles that sizes and orders choose (gmg_level_routes): the
finest rows numbered by coarse cell or by index, and the batched block sweep where a
block fits a workgroup's LDS or not, each with the bits of the other form's results."""
import sys

import numpy as np
import pytest

import synth
from tests.test_gpu_block_sweep import uneven_torus
from tests.test_gpu_parity import assert_same_bits
from tests.test_gpu_point_order import reordered

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def build(prob, **opt):
    from paper_2307_04886_amd.binding import default_options, from_problem
    return from_problem(prob, default_options(**opt))[0]


# (strided: far from one another, but the couplings of consecutive points are consecutive)
@pytest.mark.parametrize("kind,by_cell", [("grid", False), ("halves", False), ("strided", False), ("random", True)])
def test_point_order_route(kind, by_cell):
    _say(f"[gpu] route of point order {kind}")
    prob = synth.small_torus(256, 160)
    n = prob.n
    rng = np.random.default_rng(3)
    order = {"grid": np.arange(n), "random": rng.permutation(n),
             "strided": np.argsort(np.arange(n) * 7919 % n, kind="stable"),
             "halves": np.concatenate([np.arange(n // 2), n // 2 + rng.permutation(n - n // 2)])}[kind]
    gpu = build(reordered(prob, order), min_coarse_points=300)
    assert gpu.routes(0)["by_cell"] == by_cell
    assert not any(gpu.routes(l)["by_cell"] for l in range(1, gpu.num_levels))


def test_point_order_route_without_blocks():
    """Numbered by index where the next level has no blocks to order the cells by."""
    _say("[gpu] route of point order, no blocks")
    prob = synth.small_torus(256, 160)
    prob = reordered(prob, np.random.default_rng(3).permutation(prob.n))
    gpu = build(prob, min_coarse_points=300, block_min_rows=1 << 30)
    assert not gpu.routes(0)["by_cell"]


BLOCKS = {                                   # mesh, options, block in LDS in float, in double
    "cloud8": (lambda: synth.small_pointcloud(45000), dict(coarsening_ratio=0.5), True, True),
    "uneven_half": (lambda: uneven_torus(256, 200, 0.995), dict(coarsening_ratio=0.25), True, True),   # 151 KiB in double
    "uneven": (lambda: uneven_torus(256, 200, 0.995), {}, True, False),
    "cloud28": (lambda: synth.small_pointcloud(60000, 28), dict(coarsening_ratio=0.5), False, False),
}


@pytest.mark.parametrize("name", list(BLOCKS))
def test_block_route(name):
    make, opt, f32, f64 = BLOCKS[name]
    prob = make()
    gpu = build(prob, min_coarse_points=500, **opt)
    blocked = [l for l in range(gpu.num_levels) if gpu.sizes(l)["blocks"] and gpu.sizes(l)["n"] > 4096]
    assert blocked == [1]
    routes = gpu.routes(1)
    assert 0 <= routes["block_lds_f32"] <= 156 * 1024 and 0 <= routes["block_lds_f64"] <= 156 * 1024
    assert (routes["block_lds_f32"] > 0) == f32 and (routes["block_lds_f64"] > 0) == f64
    for l in set(range(gpu.num_levels)) - {1}:
        assert gpu.routes(l)["block_lds_f32"] == gpu.routes(l)["block_lds_f64"] == 0
    R = np.random.default_rng(13).uniform(-1, 1, (2, prob.n))
    for precision in ("f64", "f32"):
        _say(f"[gpu] route of blocks {name} {precision}")
        Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
        for q in range(2):
            z = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
            assert_same_bits(z, Z[q], f"{name} {precision}")


def test_routes_arguments():
    from paper_2307_04886_amd.binding import GMGError, library
    gpu = build(synth.small_torus(20, 20), min_coarse_points=100)
    for level in (-1, gpu.num_levels):
        with pytest.raises(GMGError) as e:
            gpu.routes(level)
        assert e.value.status == -1
    assert library().gmg_level_routes(gpu._h, 0, None) == -1
