"""GPU: levels swept by one workgroup whose rows are longer than the 32 entries that
it holds of a row, at the sizes where the reading of the further entries changes
shape (tiles of 16, two in flight): the oracle's bits, and the time of a phase."""
import sys
import time

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import assert_same_bits
from tests.test_gpu_pcg import PREC, both
from tests.test_gpu_small_colouring import star_of_cliques

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# the clique's rows have `clique` entries, but its last point, on the path, one more
@pytest.mark.parametrize("clique", [31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 96, 97, 129])
def test_long_rows(clique):
    prob = star_of_cliques(300, clique)
    orc, gpu = both(prob, min_coarse_points=10)
    R = np.random.default_rng(8).uniform(-1, 1, (3, prob.n))
    for precision in ("f64", "f32"):
        _say(f"[gpu] rows of {clique} entries {precision}")
        Z = gpu.precondition_batched(torch.from_numpy(R).cuda(), precision=precision).cpu().numpy()
        for q in range(3):
            zo = orc.precondition(R[q], PREC[precision])
            zg = gpu.precondition(torch.from_numpy(R[q].copy()).cuda(), precision=precision).cpu().numpy()
            assert_same_bits(zo, zg, f"{clique} {precision}")
            assert_same_bits(zo, Z[q], f"{clique} {precision} batched")
    _say(f"[gpu] rows of {clique} entries, V-cycles and new values")
    xo = orc.solve(prob.rhs, tol=0.0, max_iters=3)[0]
    xg = gpu.solve(torch.from_numpy(prob.rhs).cuda(), tol=0.0, max_iters=3)[0].cpu().numpy()
    assert_same_bits(xo, xg, f"{clique}")
    gpu.update_matrix(torch.from_numpy(prob.data).cuda())
    z2 = gpu.precondition(torch.from_numpy(R[0].copy()).cuda()).cpu().numpy()
    assert_same_bits(orc.precondition(R[0], PREC["f64"]), z2, f"{clique} updated")


def test_long_rows_grouped():
    """A group whose members' small levels have short, full and long rows."""
    from paper_2307_04886_amd.binding import default_options, from_problem, solve_pcg_grouped
    probs = [synth.small_torus(30, 20), star_of_cliques(300, 70), synth.small_pointcloud(900), synth.small_hubs(48, 40)]
    hs = [from_problem(p, default_options(min_coarse_points=60))[0] for p in probs]
    Bs = [torch.from_numpy(np.random.default_rng(9).uniform(-1, 1, (3, p.n))).cuda() for p in probs]
    for precision in ("f64", "f32"):
        _say(f"[gpu] grouped long rows {precision}")
        Xs, infos, sts, _ = solve_pcg_grouped(hs, Bs, precision=precision)
        for h, B, X, info, st in zip(hs, Bs, Xs, infos, sts):
            Y, one, s1 = h.solve_pcg_batched(B, precision=precision)
            assert st == s1 == 0
            assert_same_bits(Y.cpu().numpy(), X.cpu().numpy(), precision)
            assert [i.iterations for i in one] == [i.iterations for i in info]


@pytest.mark.parametrize("n,k", [(600, 60), (400, 100)])
def test_long_row_phase_time(n, k):
    """A phase (a colour of a sweep) of rows of 64 to 106 entries is a chain of some
    19 cycles an entry, about 1 us; reading their further entries one by one, a memory
    latency each, made it 9 to 17 us.  Bound: half of the lesser of these."""
    from paper_2307_04886_amd.binding import default_options, from_problem
    prob = synth.small_pointcloud(n, k)
    gpu, _ = from_problem(prob, default_options(min_coarse_points=50))
    phases = 4 * gpu.sizes(0)["colors"]
    r = torch.from_numpy(np.random.default_rng(10).uniform(-1, 1, prob.n)).cuda()
    z = torch.empty_like(r)
    for precision in ("f64", "f32"):
        best = float("inf")
        gpu.precondition(r, z, precision=precision)
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                gpu.precondition(r, z, precision=precision)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 10)
        _say(f"[gpu] {n} points, k = {k}, {precision}: {best * 1e6:.0f} us a cycle, {best * 1e6 / phases:.2f} us a phase")
        assert best * 1e6 / phases < 4.4


def test_long_rows_grouped_one_depth():
    """Members whose level above the coarsest has rows of up to 8, 16 and 32 entries and
    longer ones: those of up to 32 go with the longer ones."""
    from paper_2307_04886_amd.binding import default_options, from_problem, solve_pcg_grouped
    probs = [synth.small_torus(30, 20), star_of_cliques(400, 14), synth.small_pointcloud(900, 16),
             synth.small_pointcloud(800, 40), star_of_cliques(300, 30)]
    hs = [from_problem(p, default_options(max_levels=2, min_coarse_points=60))[0] for p in probs]
    longest = [int(np.diff(h.export(0, "a_rowptr")).max()) for h in hs]
    assert longest[0] <= 8 < longest[1] <= 16 < longest[2] <= 32 < longest[3] and 16 < longest[4] <= 32
    assert all(h.num_levels == 2 for h in hs)
    Bs = [torch.from_numpy(np.random.default_rng(14).uniform(-1, 1, (2, p.n))).cuda() for p in probs]
    for precision in ("f64", "f32"):
        _say(f"[gpu] grouped long rows, one depth {precision}")
        Xs, infos, sts, _ = solve_pcg_grouped(hs, Bs, precision=precision)
        for h, B, X, info, st in zip(hs, Bs, Xs, infos, sts):
            Y, one, s1 = h.solve_pcg_batched(B, precision=precision)
            assert st == s1 == 0
            assert_same_bits(Y.cpu().numpy(), X.cpu().numpy(), precision)
            assert [i.iterations for i in one] == [i.iterations for i in info]
